// bf16 GEMM on the gfx950 matrix cores for grids that do not fill the chip with 256 x 256 tiles.
//
//   ring_nt_kernel   C[M,N] = A[M,K] . B[N,K]^T (+ bias) (+ R)     both operands with the reduction index contiguous
//   share_nt_kernel  the same, the reduction of a tile shared among the waves of a workgroup
//   ring_tn_kernel   C[M,N] = sum_k At[k][m] Bt[k][n]              both operands token-major (weight gradients)
//
// With one workgroup of four waves on a compute unit nothing but the kernel itself hides the latency of a load (1-2 us
// to the memory-side cache), so what bounds these sizes is how many bytes a workgroup keeps in flight.  Operands go
// from memory straight into a ring of S LDS stages of 64 reduction indices each (global_load_lds_dwordx4, no staging
// registers); S - 1 stages are in flight while one is consumed.  A wave reads ALL fragments of the next stage while the
// MFMAs of the present one run (two register sets), so neither the LDS latency nor the barrier (one per stage) is
// exposed.  16 x 16 x 32 MFMAs with accumulators updated in place, as in the 256 x 256 kernel.  The path into LDS takes about 57 bytes a clock, which makes (BM + BN) * 128 / 57 clocks the floor of a
// stage: 575 for 128 x 128 (MFMA: 515), 431 for 128 x 64 (257), 287 for 64 x 64 (129).
#include <type_traits>

#include "common.h"

namespace mt {

namespace {

constexpr int RK = 64;         // reduction indices per stage
constexpr int kRingXcd = 8;
constexpr int kRingGroupM = 8;
typedef __attribute__((address_space(3))) void *ring_lptr;
typedef __attribute__((ext_vector_type(4))) uint32_t ru32x4;

// One load of 16 bytes per lane from base + off straight into LDS at lds + 16 lane.  Assembly because the compiler puts
// a full wait in front of every LDS read that might alias a builtin load-to-LDS; ordering is by ring_wait.
__device__ __forceinline__ void ring_load(const void *base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "s"(lds) : "memory");
}
// all but the youngest N loads of this wave have landed, its LDS reads too; then the workgroup's barrier
template <int N>
__device__ __forceinline__ void ring_wait() {
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}
template <int L, int S>
__device__ __forceinline__ void ring_wait_steps(int steps) {   // steps: wave-uniform
    if (S >= 6 && steps >= 4) ring_wait<4 * L <= 63 ? 4 * L : 0>();
    else if (S >= 5 && steps >= 3) ring_wait<3 * L <= 63 ? 3 * L : 0>();
    else if (S >= 4 && steps >= 2) ring_wait<2 * L>();
    else if (steps >= 1) ring_wait<L>();
    else ring_wait<0>();
}

// Workgroup -> tile: ids are dealt round-robin to the 8 XCDs; re-numbered so that an XCD gets a contiguous range, walked
// column by column in groups of kRingGroupM tile rows.
__device__ __forceinline__ int ring_renumber(int nb) {
    const int q = nb / kRingXcd, r = nb % kRingXcd, x = blockIdx.x % kRingXcd;
    return x * q + (x < r ? x : r) + (int)blockIdx.x / kRingXcd;
}
__device__ __forceinline__ void ring_tile(int pid, int tiles_m, int tiles_n, int *tm, int *tn) {
    const int group = kRingGroupM * tiles_n;
    const int first_m = (pid / group) * kRingGroupM;
    const int gsz = min(tiles_m - first_m, kRingGroupM);
    *tm = first_m + (pid % group) % gsz;
    *tn = (pid % group) / gsz;
}

// An fp32 tile in LDS (row pitch BN + 4; NSUM of them are added up, each BM rows after the one before) -> C, by NT threads: a store instruction
// covers whole lines, and bias, residual and accumulation read them the same way.
template <int BM, int BN, int NT, int NSUM, bool F32>
__device__ __forceinline__ void store_tile(const GemmArgs &g, const float *st, int m0, int n0) {
    constexpr int P = BN + 4;
    const int tid = threadIdx.x;
    constexpr int CPL = F32 ? 4 : 8;                  // columns per lane
    constexpr int LPR = BN / CPL, RPI = std::min(BM, NT / LPR);    // lanes per row, rows per pass
    const int r0 = tid / LPR, col = n0 + (tid % LPR) * CPL;
    if (r0 >= RPI || col >= g.N) return;
    const float *sp = st + r0 * P + (tid % LPR) * CPL;
    const auto sum = [](const float *p) {
        f32x4 v = *reinterpret_cast<const f32x4 *>(p);
#pragma unroll
        for (int k = 1; k < NSUM; ++k) v += *reinterpret_cast<const f32x4 *>(p + k * BM * P);
        return v;
    };
    // Passes in groups of U: their LDS reads, and the reads of what is added, are in flight together (a pass that ends at the last row
    // by a branch would wait for its own read); rows past the end re-read the last one and are not stored.
    constexpr int N_PASS = BM / RPI, U = N_PASS < 4 ? N_PASS : 4;
    static_assert(N_PASS % U == 0, "whole groups");
    if constexpr (F32) {
        const bool vec = !(g.ldc & 3) && !((uintptr_t)g.C & 15) && col + 4 <= g.N;
        float *cp = reinterpret_cast<float *>(g.C) + col;
        for (int it = 0; it < N_PASS; it += U) {
            if (m0 + it * RPI >= g.M) break;   // the same for the whole workgroup
            f32x4 v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = sum(sp + (it + u) * RPI * P);
            if (vec) {
                if (g.accumulate) {
                    f32x4 c[U];
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        c[u] = *reinterpret_cast<const f32x4 *>(cp + (int64_t)min(m0 + r0 + (it + u) * RPI, g.M - 1) * g.ldc);
#pragma unroll
                    for (int u = 0; u < U; ++u) v[u] += c[u];
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (m0 + r0 + (it + u) * RPI < g.M) *reinterpret_cast<f32x4 *>(cp + (int64_t)(m0 + r0 + (it + u) * RPI) * g.ldc) = v[u];
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (m0 + r0 + (it + u) * RPI >= g.M) break;
                    float *c = cp + (int64_t)(m0 + r0 + (it + u) * RPI) * g.ldc;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < g.N) c[e] = v[u][e] + (g.accumulate ? c[e] : 0.f);
                }
            }
        }
    } else {
        const int access = row_access(g.C, g.ldc, col, g.N), access_r = row_access(g.R, g.ldr, col, g.N);
        float bias[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) bias[e] = g.bias && col + e < g.N ? bf2f(g.bias[col + e]) : 0.f;
        bf16_t *cp = reinterpret_cast<bf16_t *>(g.C) + col;
        const bf16_t *rp = g.R ? g.R + col : nullptr;
        for (int it = 0; it < N_PASS; it += U) {
            if (m0 + it * RPI >= g.M) break;   // the same for the whole workgroup
            float v[U][8];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const f32x4 lo = sum(sp + (it + u) * RPI * P), hi = sum(sp + (it + u) * RPI * P + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[u][e] = lo[e] + bias[e];
                    v[u][4 + e] = hi[e] + bias[4 + e];
                }
            }
            if (rp && access_r == 16) {
                uint4 rv[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    rv[u] = *reinterpret_cast<const uint4 *>(rp + (int64_t)min(m0 + r0 + (it + u) * RPI, g.M - 1) * g.ldr);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    v[u][0] += bflo(rv[u].x); v[u][1] += bfhi(rv[u].x); v[u][2] += bflo(rv[u].y); v[u][3] += bfhi(rv[u].y);
                    v[u][4] += bflo(rv[u].z); v[u][5] += bfhi(rv[u].z); v[u][6] += bflo(rv[u].w); v[u][7] += bfhi(rv[u].w);
                }
            } else if (rp) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    row_add8(v[u], rp + (int64_t)min(m0 + r0 + (it + u) * RPI, g.M - 1) * g.ldr, access_r, col, g.N);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (m0 + r0 + (it + u) * RPI < g.M) row_store8(cp + (int64_t)(m0 + r0 + (it + u) * RPI) * g.ldc, v[u], access, col, g.N);
        }
    }
}

// The tile leaves through LDS as fp32 (the ring is free after the last stage).  A lane owns row l16 of a 16 x 16 block and its columns
// 4 hq .. + 3 (the MFMAs are issued with the operands swapped).  Row pitch BN + 4: the 16-byte writes of consecutive rows
// fall on disjoint banks.
template <int BM, int BN, int TM, int TN, bool F32>
__device__ __forceinline__ void ring_store(const GemmArgs &g, const f32x4 (&acc)[TM][TN], int m0, int n0, int wm, int wn, float *st) {
    constexpr int P = BN + 4;
    const int lane = threadIdx.x & 63, l16 = lane & 15, hq = lane >> 4;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
            *reinterpret_cast<f32x4 *>(st + (wm * TM * 16 + i * 16 + l16) * P + wn * TN * 16 + j * 16 + hq * 4) = acc[i][j];
    __syncthreads();
    store_tile<BM, BN, 256, 1, F32>(g, st, m0, n0);
}

// The walk over the stages, shared by the two kernels.  LOAD(J, T, SLOT) requests load J of stage T, READ(SET, KS, F, SLOT)
// reads fragment F of slice KS into register set SET.  Stage T lives in slot T % S.  At the top of stage T: stage T + 1
// has landed and every wave has read its fragments of stage T (one wait, one barrier), so slot T % S takes stage T + S.
// RING_NEXT() follows the loads of a stage.  RING_SEAM(t) is the next stage, t at most, in front of which RING_AT_SEAM() runs.
#define RING_STAGE(CS, NS, LOADS)                                                                       \
    {                                                                                                   \
        const int sn_ = slot + 1 == S ? 0 : slot + 1;                                                   \
        _Pragma("unroll") for (int ks = 0; ks < 2; ++ks)                                                \
            _Pragma("unroll") for (int m = 0; m < MPS; ++m) {                                           \
                constexpr int ALL = 2 * MPS;                                                            \
                const int u = ks * MPS + m;                                                             \
                if (LOADS) {                                                                            \
                    _Pragma("unroll") for (int j = u * LPS / ALL; j < (u + 1) * LPS / ALL; ++j) RING_LOAD(j, t + S, slot); \
                }                                                                                       \
                _Pragma("unroll") for (int f = m * (TM + TN) / MPS; f < (m + 1) * (TM + TN) / MPS; ++f) RING_READ(NS, ks, f, sn_); \
                const int i = m / TN, j = i & 1 ? TN - 1 - m % TN : m % TN;                             \
                mfma16_acc(acc[i][j], fr[CS][ks][TM + j], fr[CS][ks][i]);                               \
                __builtin_amdgcn_sched_barrier(0);                                                      \
            }                                                                                           \
        if (LOADS) RING_NEXT();                                                                         \
        slot = sn_;                                                                                     \
    }
#define RING_LAST_STAGE(CS, NS)                                                                         \
    {                                                                                                   \
        ring_wait_steps<LPS, S>(min(t + S - 1, nk - 1) - (t + 1));                                      \
        if (t + S < nk) {                                                                               \
            _Pragma("unroll") for (int j = 0; j < LPS; ++j) RING_LOAD(j, t + S, slot);                  \
            RING_NEXT();                                                                                \
        }                                                                                               \
        RING_STAGE(CS, NS, false);                                                                      \
    }
#define RING_WALK()                                                                                     \
    {                                                                                                   \
        ring_wait_steps<LPS, S + 1>(min(S, nk) - 1);                                                    \
        _Pragma("unroll") for (int ks = 0; ks < 2; ++ks)                                                \
            _Pragma("unroll") for (int f = 0; f < TM + TN; ++f) RING_READ(0, ks, f, 0);                 \
        int t = 0, slot = 0;                                                                            \
        const int t_end = nk - 1 - S;                                                                   \
        for (; t < t_end;) {                                                                            \
            const int stop = RING_SEAM(t_end);                                                          \
            for (; t < stop;) {                                                                         \
                ring_wait<(S - 2) * LPS>();                                                             \
                RING_STAGE(0, 1, true);                                                                 \
                ++t;                                                                                    \
                ring_wait<(S - 2) * LPS>();                                                             \
                RING_STAGE(1, 0, true);                                                                 \
                ++t;                                                                                    \
            }                                                                                           \
            RING_AT_SEAM();                                                                             \
        }                                                                                               \
        for (; t < nk;) {                                                                               \
            RING_LAST_STAGE(0, 1);                                                                      \
            if (++t == nk) break;                                                                       \
            RING_LAST_STAGE(1, 0);                                                                      \
            ++t;                                                                                        \
        }                                                                                               \
        mfma16_settle(acc);                                                                             \
    }

// LDS stage: A [BM][64] | B [BN][64] bf16, rows of 128 bytes, 16-byte chunk c of row r at position c ^ ((r >> 1) & 7)
// (conflict-free 16-byte fragment reads without padding).  TAIL (K % 64 != 0): the last, partial stage is walked first; it goes
// through registers, chunks at or beyond K as zeros.
// first >= 0: the workgroups cover the 256 x 256 tiles (tiles_m x tiles_n of them) from position `first` of that kernel's tile
// order on, each cut into (256 / BM) (256 / BN) of the tiles here.
template <int BM, int BN, int S, bool F32, bool TAIL>
__global__ __launch_bounds__(256) void ring_nt_kernel(GemmArgs g, int tiles_m, int tiles_n, int first) {
    extern __shared__ __attribute__((aligned(1024))) char ring[];
    constexpr int TM = BM / 32, TN = BN / 32, MPS = TM * TN;         // 16 x 16 blocks of a wave (2 x 2 waves)
    constexpr int LA = BM / 32, LB = BN / 32, LPS = LA + LB;         // loads of a wave per stage
    constexpr int STAGE = (BM + BN) * 128;
    static_assert(BM * (BN + 4) * 4 <= S * STAGE && S * STAGE <= 160 * 1024, "LDS");
    int tm, tn;
    if (first < 0) {
        ring_tile(ring_renumber(tiles_m * tiles_n), tiles_m, tiles_n, &tm, &tn);
    } else {
        constexpr int CM = 256 / BM, CN = 256 / BN;
        const int pid = ring_renumber((int)gridDim.x), cut = pid % (CM * CN);
        gemm_tile_of(first + pid / (CM * CN), tiles_m, tiles_n, g.group_m, &tm, &tn);
        tm = tm * CM + cut % CM;
        tn = tn * CN + cut / CM;
    }
    const int m0 = tm * BM, n0 = tn * BN;
    if (m0 >= g.M || n0 >= g.N) return;   // a cut of a ragged edge tile that lies outside
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, hq = lane >> 4;

    // wave w fills rows (BM / 4) w .. of A and (BN / 4) w .. of B, 8 rows per load; rows past the edge re-read the last one
    const bf16_t *abase = g.A + (int64_t)m0 * g.lda, *bbase = g.B + (int64_t)n0 * g.ldb;
    uint32_t off[LPS];
    const int lr = lane >> 3;
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        const int r = j < LA ? wave * (BM / 4) + j * 8 + lr : wave * (BN / 4) + (j - LA) * 8 + lr;
        const int chunk = (lane & 7) ^ ((r >> 1) & 7);
        const int row = j < LA ? min(r, g.M - 1 - m0) : min(r, g.N - 1 - n0);
        off[j] = (uint32_t)(row * (int)(j < LA ? g.lda : g.ldb) + chunk * 8) * 2u;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(ring_lptr)ring;
    const uint32_t fill_a = (uint32_t)(wave * (BM / 4) * 128), fill_b = (uint32_t)(BM * 128 + wave * (BN / 4) * 128);
    uint32_t rda[2], rdb[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const uint32_t pos = (uint32_t)(((4 * ks + hq) ^ ((l16 >> 1) & 7)) * 16);
        rda[ks] = (uint32_t)((wm * TM * 16 + l16) * 128) + pos;
        rdb[ks] = (uint32_t)(BM * 128 + (wn * TN * 16 + l16) * 128) + pos;
    }
    bf16x8 fr[2][2][TM + TN];
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nk = (g.K + RK - 1) / RK;
    // with TAIL the partial stage is walked first (below), otherwise the walk starts where the 256 x 256 kernel's does
    int kn = TAIL ? 0 : gemm_walk_start(m0 >> 8, nk) * RK;   // reduction index of the next stage to load
#define RING_NEXT()                                                                                     \
    {                                                                                                   \
        kn += RK;                                                                                       \
        if (!TAIL && kn == g.K) kn = 0;                                                                 \
    }
#define RING_LOAD(J, T, SLOT)                                                                           \
    ring_load(((J) < LA ? abase : bbase) + kn, off[J],                                                  \
              lds0 + (uint32_t)(SLOT) * STAGE + ((J) < LA ? fill_a + (J) * 1024u : fill_b + ((J) - LA) * 1024u))
#define RING_READ(SET, KS, F, SLOT)                                                                     \
    fr[SET][KS][F] = *reinterpret_cast<const bf16x8 *>(ring + (SLOT) * STAGE + ((F) < TM ? rda[KS] + (F) * 2048 : rdb[KS] + ((F) - TM) * 2048))
    ru32x4 tv[TAIL ? LPS : 1];
    const int kt = (nk - 1) * RK;
    if constexpr (TAIL) {
#pragma unroll
        for (int j = 0; j < LPS; ++j) {
            const int r = j < LA ? wave * (BM / 4) + j * 8 + lr : wave * (BN / 4) + (j - LA) * 8 + lr;
            const int chunk = (lane & 7) ^ ((r >> 1) & 7);
            const bool ok = kt + chunk * 8 < g.K;   // otherwise column 0 of the row is read (in bounds) and replaced
            const char *p = reinterpret_cast<const char *>(j < LA ? abase : bbase) + off[j] + (ok ? kt * 2 : -chunk * 16);
            tv[j] = *reinterpret_cast<const ru32x4 *>(p);
            if (!ok) tv[j] = ru32x4{0u, 0u, 0u, 0u};
        }
    } else {
#pragma unroll
        for (int j = 0; j < LPS; ++j) RING_LOAD(j, 0, 0);
        RING_NEXT();
    }
#pragma unroll
    for (int s = 1; s < S; ++s)
        if (s < nk) {
#pragma unroll
            for (int j = 0; j < LPS; ++j) RING_LOAD(j, s, s);
            RING_NEXT();
        }
    if constexpr (TAIL) {
#pragma unroll
        for (int j = 0; j < LPS; ++j)
            *reinterpret_cast<ru32x4 *>(ring + (j < LA ? fill_a + j * 1024 : fill_b + (j - LA) * 1024) + lane * 16) = tv[j];
    }
#define RING_SEAM(T) (T)
#define RING_AT_SEAM()
    RING_WALK();
#undef RING_SEAM
#undef RING_AT_SEAM
#undef RING_NEXT
#undef RING_LOAD
#undef RING_READ
    ring_store<BM, BN, TM, TN, F32>(g, acc, m0, n0, wm, wn, reinterpret_cast<float *>(ring));
}

// The ring for rows that are not whole lines (K % 64, pitches as tight as K).  A piece of 128 bytes of such a row touches two lines, and a
// line is asked for twice, by the stage that needs its beginning and by the one that needs its end: 1.14 to 1.43 times the time.  Here whole lines are
// fetched, each once, and put together when LDS is read: row r begins s_r chunks of 16 bytes behind the start of a line, so chunk c of
// stage T lies in line T + (c + s_r) / 8 of the row.  A lane's rows are 16 apart and begin alike, so that is one choice between two slots per lane,
// operand and half stage.  Chunk c + s_r of its line lies at position (c + (r >> 1)) & 7: reads are free of bank conflicts whatever s_r.
// The partial stage comes first, as in the other kernels (same order of additions, same bits): the lines are v = 0, 1 (the end of the row) and
// then 2, 3, .. (its lines 0, 1, ..), stage u = 0 (the partial one) takes lines 0 and 1, stage u > 0 lines u + 1 and u + 2.  Line v lives in slot v % S.
// At the top of stage u lines up to u + 3 have landed and every wave has read its fragments of stage u: slot (u + 1) % S takes line u + 1 + S.
// Chunks before or behind the row are replaced by ones inside, those behind are zeros in the fragments.
template <int BM, int BN, int S, bool F32>
__global__ __launch_bounds__(256) void line_nt_kernel(GemmArgs g, int tiles_m, int tiles_n) {
    extern __shared__ __attribute__((aligned(1024))) char ring[];
    constexpr int TM = BM / 32, TN = BN / 32, MPS = TM * TN;         // 16 x 16 blocks of a wave (2 x 2 waves)
    constexpr int LA = BM / 32, LB = BN / 32, LPS = LA + LB;         // loads of a wave per stage
    constexpr int STAGE = (BM + BN) * 128;
    static_assert(S >= 4 && BM * (BN + 4) * 4 <= S * STAGE && S * STAGE <= 160 * 1024, "LDS");
    int tm, tn;
    ring_tile(ring_renumber(tiles_m * tiles_n), tiles_m, tiles_n, &tm, &tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1, l16 = lane & 15, hq = lane >> 4;

    const bf16_t *abase = g.A + (int64_t)m0 * g.lda, *bbase = g.B + (int64_t)n0 * g.ldb;
    const int nk = (g.K + RK - 1) / RK, nv = nk > 1 ? nk + 2 : 2;
    const auto start_of = [&](bool a, int row) { return (int)(((uintptr_t)(a ? abase : bbase) >> 4) + (uint32_t)row * (uint32_t)((a ? g.lda : g.ldb) >> 3)) & 7; };
    // wave w fills rows (BM / 4) w .. of A and (BN / 4) w .. of B, 8 rows per load; rows past the edge re-read the last one
    uint32_t off[LPS];   // from 128 bytes in front of a line 0
    const auto row_of = [&](int j) { return j < LA ? wave * (BM / 4) + j * 8 + (lane >> 3) : wave * (BN / 4) + (j - LA) * 8 + (lane >> 3); };
    const auto row_off = [&](int j) {
        return (uint32_t)((j < LA ? min(row_of(j), g.M - 1 - m0) : min(row_of(j), g.N - 1 - n0)) * (int)(j < LA ? g.lda : g.ldb)) * 2u;
    };
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        const int r = row_of(j), s = start_of(j < LA, r);
        off[j] = row_off(j) + 128u + (((lane - (r >> 1) + s) & 7) - s) * 16u;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(ring_lptr)ring;
    const uint32_t fill_a = (uint32_t)(wave * (BM / 4) * 128), fill_b = (uint32_t)(BM * 128 + wave * (BN / 4) * 128);
    uint32_t rda[2], rdb[2];
    bool ca[2], cb[2];   // the chunk lies in the second line
    {
        const int sa = start_of(true, wm * TM * 16 + l16), sb = start_of(false, wn * TN * 16 + l16);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const uint32_t pos = (uint32_t)(((4 * ks + hq + (l16 >> 1)) & 7) * 16);
            rda[ks] = (uint32_t)((wm * TM * 16 + l16) * 128) + pos;
            rdb[ks] = (uint32_t)(BM * 128 + (wn * TN * 16 + l16) * 128) + pos;
            ca[ks] = 4 * ks + hq + sa >= 8;
            cb[ks] = 4 * ks + hq + sb >= 8;
        }
    }
    bf16x8 fr[2][2][TM + TN];
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const auto load = [&](int j, int line, int slot) {   // a line in the middle of the rows: 0 < line < nk - 1
        ring_load((j < LA ? abase : bbase) + (line - 1) * 64, off[j], lds0 + (uint32_t)slot * STAGE + (j < LA ? fill_a + j * 1024u : fill_b + (j - LA) * 1024u));
    };
    const auto load_any = [&](int line, int slot) {
#pragma unroll
        for (int j = 0; j < LPS; ++j) {
            const int first = (int)row_off(j), at = (int)off[j] + (line - 1) * 128;
            ring_load(j < LA ? abase : bbase, (uint32_t)min(max(at, first), first + (g.K - 8) * 2),
                      lds0 + (uint32_t)slot * STAGE + (j < LA ? fill_a + j * 1024u : fill_b + (j - LA) * 1024u));
        }
    };
    const auto line_of = [&](int v) { return v < 2 ? nk - 1 + v : v - 2; };
    uint32_t ra[2], rb[2];
    const auto aim = [&](int slot) {   // the reads of the stage whose first line is in this slot
        const uint32_t lo = (uint32_t)slot * STAGE, hi = (uint32_t)(slot + 1 == S ? 0 : slot + 1) * STAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            ra[ks] = rda[ks] + (ca[ks] ? hi : lo);
            rb[ks] = rdb[ks] + (cb[ks] ? hi : lo);
        }
    };
    const auto read = [&](auto set, int ks, int f) {
        fr[set()][ks][f] = *reinterpret_cast<const bf16x8 *>(ring + (f < TM ? ra[ks] + f * 2048 : rb[ks] + (f - TM) * 2048));
    };
    const auto next = [&](int slot) { return slot + 1 == S ? 0 : slot + 1; };

#pragma unroll
    for (int v = 0; v < S; ++v)
        if (v < nv) load_any(line_of(v), v);
    ring_wait_steps<LPS, S + 1>(min(S, nv) - 2);
    aim(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const bool there = (nk - 1) * RK + (4 * ks + hq) * 8 < g.K;
#pragma unroll
        for (int f = 0; f < TM + TN; ++f) {
            read(std::integral_constant<int, 0>(), ks, f);
            ru32x4 w = __builtin_bit_cast(ru32x4, fr[0][ks][f]);
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = there ? w[e] : 0u;
            fr[0][ks][f] = __builtin_bit_cast(bf16x8, w);
        }
    }
    mfma16_begin(acc);
    int u = 0, slot = 1;   // slot: (u + 1) % S, what is free at the top of stage u
    // the products of stage u, the fragments of the next one, and line u + 1 + S if it lies in the middle of the rows
    const auto stage = [&](auto set, auto loads) {
        constexpr int C = set();
        aim(next(slot));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int m = 0; m < MPS; ++m) {
                const int w = ks * MPS + m;
                if constexpr (loads()) {
#pragma unroll
                    for (int j = w * LPS / (2 * MPS); j < (w + 1) * LPS / (2 * MPS); ++j) load(j, u + S - 1, slot);
                }
#pragma unroll
                for (int f = m * (TM + TN) / MPS; f < (m + 1) * (TM + TN) / MPS; ++f) read(std::integral_constant<int, 1 - C>(), ks, f);
                const int i = m / TN, j = i & 1 ? TN - 1 - m % TN : m % TN;
                mfma16_acc(acc[i][j], fr[C][ks][TM + j], fr[C][ks][i]);
                __builtin_amdgcn_sched_barrier(0);
            }
        slot = next(slot);
        ++u;
    };
    const auto last_stage = [&](auto set) {
        ring_wait_steps<LPS, S>(min(u == 0 ? S - 1 : u + S, nv - 1) - (u + 3));
        if (u == 0 && S < nv) load_any(line_of(S), 0);
        if (u + 1 + S < nv) load_any(line_of(u + 1 + S), slot);
        stage(set, std::false_type());
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    last_stage(even);
    const int whole = nv - 2 - S;   // stages below this one load lines in the middle
    while (u + 1 < whole) {
        ring_wait<(S - 3) * LPS>();
        stage(odd, std::true_type());
        ring_wait<(S - 3) * LPS>();
        stage(even, std::true_type());
    }
    while (u < nk) {
        last_stage(odd);
        if (u == nk) break;
        last_stage(even);
    }
    mfma16_settle(acc);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    ring_store<BM, BN, TM, TN, F32>(g, acc, m0, n0, wm, wn, reinterpret_cast<float *>(ring));
}

// LDS stage: A [64][BM] | B [64][BN] bf16 as in memory; fragments are read with the transposing load: lane (hq, i) supplies k
// row 8 hq + (i >> 2) (and + 4) of the 32-row slice, 8 bytes at column 4 (i & 3) of the block's 16.  Half a wave reads rows 0 .. 3
// and 8 .. 11, 32 bytes each: 32-byte column group c of row r sits at group position c ^ ring_swz(r), which puts those
// eight on disjoint banks.  A wave-load fills 1024 / (2 BM) rows.  The token range may be split over workgroups (g.split_k).
template <int W>
__device__ __forceinline__ int ring_swz(int r) { return ((W == 64 ? (r >> 1) & 1 : r & 3) << 1) | ((r >> 3) & 1); }

// CHAINS: at most `chain` stages (even) are added up in one go; the sums so far are kept in a second set of registers.
template <int BM, int BN, int S, bool CHAINS>
__global__ __launch_bounds__(256) void ring_tn_kernel(GemmArgs g, int tiles_m, int tiles_n, int chain) {
    extern __shared__ __attribute__((aligned(1024))) char ring[];
    typedef __attribute__((address_space(3))) s16x4 *trptr;
    constexpr int TM = BM / 32, TN = BN / 32, MPS = TM * TN;
    constexpr int LA = BM / 32, LB = BN / 32, LPS = LA + LB;
    constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
    static_assert(BM * (BN + 4) * 4 <= S * STAGE && S * STAGE <= 160 * 1024, "LDS");
    const int n_tiles = tiles_m * tiles_n;
    int pid = ring_renumber(n_tiles * g.split_k);
    const int chunk = pid / n_tiles;
    pid -= chunk * n_tiles;
    const int nk_all = g.K / RK;
    const int kb = (int)((int64_t)chunk * nk_all / g.split_k), nk = (int)((int64_t)(chunk + 1) * nk_all / g.split_k) - kb;
    if (chunk > 0) {
        g.C = g.split_ws + (int64_t)(chunk - 1) * g.M * g.N;
        g.ldc = g.N;
        g.accumulate = 0;
    }
    int tm, tn;
    ring_tile(pid, tiles_m, tiles_n, &tm, &tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    const bf16_t *abase = g.A + (int64_t)kb * RK * g.lda, *bbase = g.B + (int64_t)kb * RK * g.ldb;   // of the next stage to load
    const int64_t astep = (int64_t)RK * g.lda, bstep = (int64_t)RK * g.ldb;
    uint32_t off[LPS];
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        // lane l delivers to 16-byte position l % (W / 8) of its row and fetches the chunk that belongs there; chunks
        // past the edge re-read the last one
        constexpr int PA = BM / 8, PB = BN / 8;
        if (j < LA) {
            const int r = wave * 16 + j * (64 / PA) + lane / PA, p = lane % PA;
            const int c = (((p >> 1) ^ ring_swz<BM>(r)) << 1) | (p & 1);
            off[j] = (uint32_t)(r * (int)g.lda + min(m0 + c * 8, g.M - 8)) * 2u;
        } else {
            const int r = wave * 16 + (j - LA) * (64 / PB) + lane / PB, p = lane % PB;
            const int c = (((p >> 1) ^ ring_swz<BN>(r)) << 1) | (p & 1);
            off[j] = (uint32_t)(r * (int)g.ldb + min(n0 + c * 8, g.N - 8)) * 2u;
        }
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(ring_lptr)ring;
    const uint32_t fill_a = (uint32_t)(wave * 16 * BM * 2), fill_b = (uint32_t)(A_BYTES + wave * 16 * BN * 2);
    uint32_t rd[TM + TN];
    {
        const int i = lane & 15, row = (lane >> 4) * 8 + (i >> 2), inner = (i & 3) * 8;
#pragma unroll
        for (int f = 0; f < TM + TN; ++f)
            rd[f] = f < TM ? (uint32_t)(row * BM * 2 + ((wm * TM + f) ^ ring_swz<BM>(row)) * 32 + inner)
                           : (uint32_t)(A_BYTES + row * BN * 2 + ((wn * TN + f - TM) ^ ring_swz<BN>(row)) * 32 + inner);
    }
    bf16x8 fr[2][2][TM + TN];
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

#define RING_NEXT()                                                                                     \
    {                                                                                                   \
        abase += astep;                                                                                 \
        bbase += bstep;                                                                                 \
    }
#define RING_LOAD(J, T, SLOT)                                                                           \
    ring_load((J) < LA ? abase : bbase, off[J],                                                         \
              lds0 + (uint32_t)(SLOT) * STAGE + ((J) < LA ? fill_a + (J) * 1024u : fill_b + ((J) - LA) * 1024u))
#define RING_READ(SET, KS, F, SLOT)                                                                     \
    {                                                                                                   \
        const int ROW_ = 2 * ((F) < TM ? BM : BN);                                                  \
        const char *p_ = ring + (SLOT) * STAGE + rd[F] + (KS) * 32 * ROW_;                              \
        const s16x4 lo_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((trptr)(p_));                         \
        const s16x4 hi_ = __builtin_amdgcn_ds_read_tr16_b64_v4i16((trptr)(p_ + 4 * ROW_));              \
        typedef __attribute__((ext_vector_type(8))) short s16x8_;                                       \
        const s16x8_ v_ = {lo_[0], lo_[1], lo_[2], lo_[3], hi_[0], hi_[1], hi_[2], hi_[3]};             \
        fr[SET][KS][F] = __builtin_bit_cast(bf16x8, v_);                                                \
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (s < nk) {
#pragma unroll
            for (int j = 0; j < LPS; ++j) RING_LOAD(j, s, s);
            RING_NEXT();
        }
    f32x4 sum[CHAINS ? TM : 1][TN];
#define RING_ADD_CHAIN()                                                                                \
    {                                                                                                   \
        _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                  \
            _Pragma("unroll") for (int j = 0; j < TN; ++j) sum[i][j] += acc[i][j];                      \
    }
#define RING_SEAM(T) (CHAINS ? min(seam, (T)) : (T))
#define RING_AT_SEAM()                                                                                  \
    if (CHAINS && t == seam) {                                                                          \
        mfma16_settle(acc);                                                                             \
        RING_ADD_CHAIN();                                                                               \
        _Pragma("unroll") for (int i = 0; i < TM; ++i)                                                  \
            _Pragma("unroll") for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};       \
        seam += chain;                                                                                  \
    }
    int seam = chain;
    if constexpr (CHAINS) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    RING_WALK();
#undef RING_SEAM
#undef RING_AT_SEAM
#undef RING_NEXT
#undef RING_LOAD
#undef RING_READ
    if constexpr (CHAINS) {
        RING_ADD_CHAIN();
        ring_store<BM, BN, TM, TN, true>(g, sum, m0, n0, wm, wn, reinterpret_cast<float *>(ring));
        return;
    }
#undef RING_ADD_CHAIN
    ring_store<BM, BN, TM, TN, true>(g, acc, m0, n0, wm, wn, reinterpret_cast<float *>(ring));
}

// Few tiles and a long reduction: the ring above walks it stage after stage (0.26 us each with 64 x 64 tiles) while most of the chip idles, and every
// stage waits for the slowest of four waves.  Here the NW waves of a workgroup share the reduction of a tile: wave w multiplies the stages w, w + NW, ...
// out of a ring of S stages of its own, which it fills and waits for without its neighbours; the sums are added in LDS, in order.  Together the rings
// hold what LDS does: 128 KB in flight, 96 for 32 x 64 and 128 x 64 (whose accumulators leave room for four waves).  What bounds it is the path of a
// compute unit for loads, (BM + BN) * 128 / 57 clocks a stage, and with most of the chip at work what an XCD can fetch beyond its L2.
// us, operands from memory, before -> now: 200 x 128 x 10880 40 -> 17 (32 x 32 tiles, eight waves), 400 x 1088 x 17216 94 -> 47 (32 x 64, eight),
// 1248 x 648 x 7040 41 -> 28 (64 x 64, four), 1992 x 864 x 17232 161 -> 134 (128 x 64, four).
// A partial last stage (K % 64) belongs to the wave whose turn it is, first; it goes through registers, chunks at or beyond K as zeros.
template <int TM, int TN, int NW, int S>
struct ShareLds {
    static constexpr uint32_t STAGE = 16 * (TM + TN) * 128, SUM = 16 * TM * (16 * TN + 4) * sizeof(float), BYTES = NW * std::max(S * STAGE, SUM);
};
template <int TM, int TN, int NW, int S, bool F32>
__global__ __launch_bounds__(64 * NW) void share_nt_kernel(GemmArgs g, int tiles_m, int tiles_n) {
    extern __shared__ __attribute__((aligned(1024))) char ring[];
    constexpr int BM = 16 * TM, BN = 16 * TN, P = BN + 4, LA = BM / 8, LPS = (BM + BN) / 8;
    constexpr uint32_t STAGE = ShareLds<TM, TN, NW, S>::STAGE;
    int tm, tn;
    ring_tile(ring_renumber(tiles_m * tiles_n), tiles_m, tiles_n, &tm, &tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, hq = lane >> 4;
    const bf16_t *abase = g.A + (int64_t)m0 * g.lda, *bbase = g.B + (int64_t)n0 * g.ldb;
    // a load covers 8 rows of 128 bytes, in the layout of the ring above; rows past the edge re-read the last one
    uint32_t off[LPS];
#pragma unroll
    for (int j = 0; j < LPS; ++j) {
        const int r = (j < LA ? j : j - LA) * 8 + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
        off[j] = (uint32_t)((j < LA ? min(r, g.M - 1 - m0) * (int)g.lda : min(r, g.N - 1 - n0) * (int)g.ldb) + chunk * 8) * 2u;
    }
    char *const mine = ring + wave * (S * STAGE);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(ring_lptr)ring + wave * (S * STAGE);
    uint32_t rd[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) rd[ks] = (uint32_t)(l16 * 128 + (((4 * ks + hq) ^ ((l16 >> 1) & 7)) << 4));
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const auto request = [&](int i, int slot) {   // this wave's i-th stage
        const int kn = (wave + i * NW) * RK;
#pragma unroll
        for (int j = 0; j < LPS; ++j) ring_load((j < LA ? abase : bbase) + kn, off[j], lds0 + slot * STAGE + j * 1024u);
    };
    bf16x8 fr[2][TM + TN];
    const auto read = [&](int slot) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int f = 0; f < TM + TN; ++f) fr[ks][f] = *reinterpret_cast<const bf16x8 *>(mine + slot * STAGE + rd[ks] + f * 2048);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (the slot is free)
    };
    const auto multiply = [&]() {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int jj = i & 1 ? TN - 1 - j : j;
                    mfma16_acc(acc[i][jj], fr[ks][TM + jj], fr[ks][i]);
                }
    };
    const int whole = g.K / RK, n = (whole - wave + NW - 1) / NW;
    if (g.K % RK && wave == whole % NW) {
#pragma unroll
        for (int j = 0; j < LPS; ++j) {
            const int r = (j < LA ? j : j - LA) * 8 + (lane >> 3), chunk = (lane & 7) ^ ((r >> 1) & 7);
            const bool ok = whole * RK + chunk * 8 < g.K;   // otherwise column 0 of the row is read (in bounds) and replaced
            ru32x4 v = *reinterpret_cast<const ru32x4 *>(reinterpret_cast<const char *>(j < LA ? abase : bbase) + off[j] + (ok ? whole * (RK * 2) : -chunk * 16));
            if (!ok) v = ru32x4{0u, 0u, 0u, 0u};
            *reinterpret_cast<ru32x4 *>(mine + j * 1024 + lane * 16) = v;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        read(0);
        multiply();
        mfma16_drain();
    }
#pragma unroll
    for (int s = 0; s < S; ++s)
        if (s < n) request(s, s);
    int slot = 0;
    for (int i = 0; i < n; ++i) {
        if (i + S <= n) asm volatile("s_waitcnt vmcnt(%0)" : : "n"((S - 1) * LPS) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        read(slot);
        if (i + S < n) request(i + S, slot);
        multiply();
        slot = slot + 1 == S ? 0 : slot + 1;
    }
    mfma16_settle(acc);
    __syncthreads();
    float *sum = reinterpret_cast<float *>(ring) + wave * (BM * P) + l16 * P + hq * 4;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4 *>(sum + i * 16 * P + j * 16) = acc[i][j];
    __syncthreads();
    store_tile<BM, BN, 64 * NW, NW, F32>(g, reinterpret_cast<float *>(ring), m0, n0);
}
template <int TM, int TN, int NW, int S, bool F32>
hipError_t launch_share_one(const GemmArgs &g, hipStream_t s) {
    static std::atomic<bool> attr{false};
    constexpr size_t lds = ShareLds<TM, TN, NW, S>::BYTES;
    static_assert(lds <= 160 * 1024, "LDS");
    const hipError_t e = ensure_lds(share_nt_kernel<TM, TN, NW, S, F32>, lds, &attr);
    if (e != hipSuccess) return e;
    const int tiles_m = (g.M + 16 * TM - 1) / (16 * TM), tiles_n = (g.N + 16 * TN - 1) / (16 * TN);
    hipLaunchKernelGGL((share_nt_kernel<TM, TN, NW, S, F32>), dim3((unsigned)(tiles_m * tiles_n)), dim3(64 * NW), lds, s, g, tiles_m, tiles_n);
    return hipGetLastError();
}
template <int TM, int TN, int NW, int S>
hipError_t launch_share(const GemmArgs &g, hipStream_t s) {
    return g.out_fp32 ? launch_share_one<TM, TN, NW, S, true>(g, s) : launch_share_one<TM, TN, NW, S, false>(g, s);
}

template <int BM, int BN, int S, bool F32, bool TAIL>
hipError_t launch_nt_one(const GemmArgs &g, int first, hipStream_t s) {
    static std::atomic<bool> attr{false};
    constexpr size_t lds = (size_t)S * (BM + BN) * 128;
    const hipError_t e = ensure_lds(ring_nt_kernel<BM, BN, S, F32, TAIL>, lds, &attr);
    if (e != hipSuccess) return e;
    const int bm = first < 0 ? BM : 256, bn = first < 0 ? BN : 256;
    const int tiles_m = (g.M + bm - 1) / bm, tiles_n = (g.N + bn - 1) / bn;
    const int blocks = first < 0 ? tiles_m * tiles_n : (tiles_m * tiles_n - first) * (256 / BM) * (256 / BN);
    hipLaunchKernelGGL((ring_nt_kernel<BM, BN, S, F32, TAIL>), dim3((unsigned)blocks), dim3(256), lds, s, g, tiles_m, tiles_n, first);
    return hipGetLastError();
}
template <int BM, int BN, int S, bool F32>
hipError_t launch_line_one(const GemmArgs &g, hipStream_t s) {
    static std::atomic<bool> attr{false};
    constexpr size_t lds = (size_t)S * (BM + BN) * 128;
    const hipError_t e = ensure_lds(line_nt_kernel<BM, BN, S, F32>, lds, &attr);
    if (e != hipSuccess) return e;
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    hipLaunchKernelGGL((line_nt_kernel<BM, BN, S, F32>), dim3((unsigned)(tiles_m * tiles_n)), dim3(256), lds, s, g, tiles_m, tiles_n);
    return hipGetLastError();
}
template <int BM, int BN, int S>
hipError_t launch_line(const GemmArgs &g, hipStream_t s) {
    return g.out_fp32 ? launch_line_one<BM, BN, S, true>(g, s) : launch_line_one<BM, BN, S, false>(g, s);
}
template <int BM, int BN, int S>
hipError_t launch_nt(const GemmArgs &g, int first, hipStream_t s) {
    if (g.K % RK) return g.out_fp32 ? launch_nt_one<BM, BN, S, true, true>(g, first, s) : launch_nt_one<BM, BN, S, false, true>(g, first, s);
    return g.out_fp32 ? launch_nt_one<BM, BN, S, true, false>(g, first, s) : launch_nt_one<BM, BN, S, false, false>(g, first, s);
}
template <int BM, int BN, int S, bool CHAINS>
hipError_t launch_tn_one(const GemmArgs &g, int chain, hipStream_t s) {
    static std::atomic<bool> attr{false};
    constexpr size_t lds = (size_t)S * (BM + BN) * 128;
    const hipError_t e = ensure_lds(ring_tn_kernel<BM, BN, S, CHAINS>, lds, &attr);
    if (e != hipSuccess) return e;
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    hipLaunchKernelGGL((ring_tn_kernel<BM, BN, S, CHAINS>), dim3((unsigned)(tiles_m * tiles_n * g.split_k)), dim3(256), lds, s, g,
                       tiles_m, tiles_n, chain);
    return hipGetLastError();
}
// partial_sums: of every output, in all
template <int BM, int BN, int S>
hipError_t launch_tn(const GemmArgs &g, int partial_sums, hipStream_t s) {
    const int chains = (partial_sums + g.split_k - 1) / g.split_k, stages = g.K / RK / g.split_k, chain = stages / chains & ~1;
    return chains > 1 && chain > 0 ? launch_tn_one<BM, BN, S, true>(g, chain, s) : launch_tn_one<BM, BN, S, false>(g, 0, s);
}

}  // namespace

// Three stages each: a fourth or fifth measured the same (4096^3: 118.6, 119.5, 120.6 us with 128 x 128 tiles), and three
// of 24 or 16 KB let two or three workgroups share a compute unit.
hipError_t gemm_nt_ring(const GemmArgs &g, RingTile tile, int first, hipStream_t s) {
    switch (tile) {
        case RingTile::t256x128: return launch_nt<256, 128, 3>(g, first, s);
        case RingTile::t128x128: return launch_nt<128, 128, 3>(g, first, s);
        case RingTile::t128x64: return launch_nt<128, 64, 3>(g, first, s);
        case RingTile::t64x64: return launch_nt<64, 64, 3>(g, first, s);
        case RingTile::l128x128: return launch_line<128, 128, 5>(g, s);
        case RingTile::l128x64: return launch_line<128, 64, 6>(g, s);
        case RingTile::l64x64: return launch_line<64, 64, 5>(g, s);
        case RingTile::s128x64: return launch_share<8, 4, 4, 1>(g, s);
        case RingTile::s64x64: return launch_share<4, 4, 4, 2>(g, s);
        case RingTile::s32x64: return launch_share<2, 4, 8, 1>(g, s);
        case RingTile::s32x32: return launch_share<2, 2, 8, 2>(g, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t gemm_tn_ring(const GemmArgs &g, RingTile tile, int partial_sums, hipStream_t s) {
    switch (tile) {
        case RingTile::t256x128: return launch_tn<256, 128, 3>(g, partial_sums, s);
        case RingTile::t128x128: return launch_tn<128, 128, 3>(g, partial_sums, s);
        case RingTile::t128x64: return launch_tn<128, 64, 3>(g, partial_sums, s);
        case RingTile::t64x64: return launch_tn<64, 64, 3>(g, partial_sums, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mt
