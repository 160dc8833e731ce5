// Causal flash attention for gfx950, forward and backward, grouped KV heads.
//
// The attention inside f_i and LocalBackward (Algorithm 1) never materialises the
// T x T score matrix: scores are produced tile by tile on the matrix cores, the
// softmax is carried online (running maximum and sum per query), and the backward
// recomputes the probabilities from the saved log-sum-exp.
//
// Register layout.  v_mfma_f32_32x32x16_bf16 leaves, in lane l, the column l%32 of
// the 32x32 result with rows 8(r/4) + 4(l/32) + r%4 for r = 0..15.  The kernels are
// arranged so that the "column" is always the index a wave owns:
//
//   forward, dQ kernel:  S^T = K Q^T, so a lane owns one query.  Row statistics
//       (max, sum, lse, delta) are per-lane scalars; the only cross-lane step is one
//       exchange with lane l^32.  P^T in registers is already a valid B operand for
//       O^T = V^T P^T and dQ^T = K^T dS^T (the reduction index of an MFMA may be
//       permuted freely as long as both operands use the same permutation).
//   dK/dV kernel:        S = Q K^T, so a lane owns one key; dV^T = dO^T P and
//       dK^T = Q^T dS take P and dS from registers in the same way.
//
// The A operands of those second products (V^T, K^T, dO^T, Q^T) are never built in memory:
// they are read from the natural row-major LDS tiles with the gfx950 transposing LDS read
// (ds_read_b64_tr_b16), which hands each lane four consecutive rows of one column; two such
// reads give exactly the eight reduction indices of the accumulator permutation.
// dQ and dK/dV walk the scores apart, in kernels of their own or side by side in one launch (small problems): no atomics, results are bit-reproducible.
//
// Tiles go from memory to LDS without passing through registers (DirectTile); where their 16-byte chunks lie is chosen so that
// row-wise and transposing reads are free of bank conflicts.  Against tiles that were fetched into registers and written to LDS
// (rows padded by 80 bytes): forward 2-15 %, backward 4-19 % faster, most on short walks.
#include <algorithm>
#include <numeric>

#include "common.h"

namespace mt {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kLazyMax = 8.0f;  // forward: the running maximum may lag the true one by this much (log2 units)

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// Unpadded LDS tiles, filled by loads that write LDS directly (a wave's 64 lanes x 16 bytes land one after the other, so padding is
// not possible): the 16-byte chunk c of row r lies at position c ^ swz(r) of its row, and every lane fetches the chunk that belongs at its
// position.  swz takes different values for the rows that one pass of a 16-byte row read covers (16 rows of 256 bytes, 8 pairs of rows
// of 128 bytes), and different 64-byte groups for the four rows of a transposing read: both are free of bank conflicts.
template <int HD>
__device__ __forceinline__ int swz(int r) {
    return HD == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : ((r & 2) << 1) | ((r >> 2) & 3);
}
// byte offset of the lane's part of a row-wise fragment (row l32, 8 columns from 8 hl): k-step ks lies at row_off ^ (32 ks), rows + 32 n at + n 64 HD
template <int HD>
__device__ __forceinline__ uint32_t row_off(int l32, int hl) { return l32 * (2 * HD) + ((hl ^ swz<HD>(l32)) << 4); }
// The same for a transposing fragment read: columns + 32 hb at off ^ (64 hb), rows + 8 at + 16 HD and ^ 32.  Its result is the A operand
// of an MFMA whose output rows are the tile's columns 32 hb .. + 31 (lane l % 32 <-> column) and whose eight reduction slots of lane
// half hl are the rows row0 + 4 hl + {0..3} and row0 + 8 + 4 hl + {0..3}: the order in which a lane holds the matching accumulator
// registers of a 32x32 block.  ds_read_b64_tr_b16 works on groups of 16 lanes: lane i of a group supplies the address of 4
// consecutive columns of one row (i / 4); it receives column i of the 4 x 16 block so formed, rows 0..3.
template <int HD>
__device__ __forceinline__ uint32_t tr_off_swz(int lane) {
    const int g = lane >> 4, i = lane & 15, r = (g >> 1) * 4 + (i >> 2);
    return r * (2 * HD) + ((((g & 1) * 2 + ((i & 3) >> 1)) ^ swz<HD>(r)) << 4) + (i & 1) * 8;
}
template <int HD>
__device__ __forceinline__ bf16x8 read_tr_swz(const char *tile, uint32_t off, int row0, int hb) {
    typedef __attribute__((address_space(3))) s16x4 *lds_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(tile + (off ^ (hb * 64)) + row0 * (2 * HD)));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(tile + (off ^ (hb * 64) ^ 32) + (row0 + 8) * (2 * HD)));
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
}
__host__ __device__ inline bool near_pitch(int64_t ld) { return ld >= 0 && ld < ((int64_t)1 << 27); }
// Fills such a tile of ROWS rows with the rows row0 .. of src (pitch ld), NW waves.  The loads are assembly and the waits for them are
// written by hand: in front of every LDS read that might alias a builtin load-to-LDS the compiler waits for all of them.  A load covers
// 4 or 8 whole rows, rows come in multiples of 8, so rows past the end (row_end) are replaced by the last ones for a whole load at a
// time, in scalar registers.  The lane's offset from the first row of a load has 32 bits; FAR: row pitches beyond that, or negative, a
// 64-bit address per lane.
template <int ROWS, int HD, int NW, bool FAR, int GS = 1024>
struct DirectTile {
    static constexpr int LPR = HD / 8, RPL = 64 / LPR, N = ROWS / (RPL * NW);   // lanes per row, rows per load, loads of a wave
    static_assert(N * RPL * NW == ROWS, "tile must split evenly over the waves");
    uint32_t row_bytes, chunk, lds_wave;
    int r, wave;
    __device__ __forceinline__ void init(const void *smem, int64_t ld, int lane, int wave_) {
        typedef __attribute__((address_space(3))) const void *lptr;
        wave = wave_;
        r = lane / LPR;
        row_bytes = r * (uint32_t)ld * 2;
        chunk = ((lane % LPR) ^ (GS == 1024 ? swz<HD>(RPL * wave_ + r) : r << 2)) << 4;
        lds_wave = (uint32_t)(uintptr_t)(lptr)smem + (uint32_t)wave_ * GS;
    }
    __device__ __forceinline__ void load(uint32_t lds_off, const bf16_t *src, int64_t ld, int row0, int row_end) const {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int row = min(row0 + RPL * (wave + NW * j), row_end - RPL);
            const bf16_t *p = src + (int64_t)row * ld;
            const uint32_t m0 = lds_wave + lds_off + j * (NW * GS);
            const uint32_t c = GS == 1024 && RPL * NW % 16 ? chunk ^ (swz<HD>(RPL * NW * j) << 4) : chunk;   // (the rows of a load differ from those of the first)
            if (!FAR) {
                asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(row_bytes + c), "s"(p), "s"(m0) : "memory");
            } else {
                const char *q = reinterpret_cast<const char *>(p + (int64_t)r * ld) + c;
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(q), "s"(m0) : "memory");
            }
        }
    }
    // the pieces that this lane delivers, into registers instead
    __device__ __forceinline__ void load_to(u32x4 (&v)[N], const bf16_t *src, int64_t ld, int row0, int row_end) const {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const bf16_t *p = src + (int64_t)min(row0 + RPL * (wave + NW * j), row_end - RPL) * ld;
            const uint32_t c = GS == 1024 && RPL * NW % 16 ? chunk ^ (swz<HD>(RPL * NW * j) << 4) : chunk;
            v[j] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(p) + (FAR ? (int64_t)r * ld * 2 : row_bytes) + c);
        }
    }
};
// (in a scalar register: what depends on it is a scalar branch)
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
__device__ __forceinline__ float scalar(float v) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))); }
// all tiles that this wave asked for have landed and its LDS reads are done, and so have those of the other waves
// The first wait is one that the compiler understands: otherwise it waits inside the loop for the loads of the fragments in front of it,
// over and over, and with them for the tile that has just been asked for.
__device__ __forceinline__ void tile_barrier() {
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ uint32_t lds_address(const void *smem) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)smem; }
// Tiles of the backward.  It reads most of them row-wise and transposed and has fewer registers for addresses, so with head_dim 128 the
// four rows of a load are followed by 16 bytes of padding and only a chunk's 64-byte group is swizzled (by the row's place in its load:
// the rows of a load then differ in the group, the loads in the place within it): the other column bits, and all row steps, are constants of
// the instruction.  head_dim 64: as above.
template <int HD>
struct BwdTile {
    static constexpr int GS = HD == 128 ? 1040 : 1024, RPL = 512 / HD, ROW = 2 * HD;
    static constexpr uint32_t BYTES = 64 / RPL * GS;   // of 64 rows
    static __host__ __device__ constexpr uint32_t rows(int n) { return n / RPL * GS; }   // offset of row n (a multiple of 8)
    uint32_t ra[4], ta[HD / 32];   // (LDS addresses as numbers: through a pointer to the dynamic LDS the compiler adds its base, 0, over and over)
    __device__ __forceinline__ void init(const void *smem, int lane) {
        const uint32_t base = lds_address(smem);
        const int l32 = lane & 31, hl = lane >> 5, g = lane >> 4, i = lane & 15;
#pragma unroll
        for (int n = 0; n < 4; ++n)
            ra[n] = base + (HD == 128 ? l32 / 4 * GS + (l32 & 3) * ROW + ((n ^ (l32 & 3)) << 6) + hl * 16 : l32 * ROW + (((2 * n + hl) ^ swz<HD>(l32)) << 4));
        const int r = (g >> 1) * 4 + (i >> 2);
#pragma unroll
        for (int hb = 0; hb < HD / 32; ++hb)
            ta[hb] = base + (HD == 128 ? (g >> 1) * GS + (i >> 2) * ROW + ((hb ^ (i >> 2)) << 6) + (g & 1) * 32 + (i & 3) * 8
                               : r * ROW + (((hb * 4 + (g & 1) * 2 + ((i & 3) >> 1)) ^ swz<HD>(r)) << 4) + (i & 1) * 8);
        // (one register each: known too well they are taken apart, and every combination with a constant is kept)
#pragma unroll
        for (int n = 0; n < 4; ++n) asm volatile("" : "+v"(ra[n]));
#pragma unroll
        for (int hb = 0; hb < HD / 32; ++hb) asm volatile("" : "+v"(ta[hb]));
    }
    // 8 columns from 16 ks + 8 hl on of the lane's row (l32; add rows(n) to the tile's address for row n + l32)
    __device__ __forceinline__ bf16x8 row_frag(uint32_t tile, int ks) const {
        typedef __attribute__((address_space(3))) const bf16x8 *lds_ptr;
        return *(lds_ptr)(tile + (HD == 128 ? ra[ks >> 1] + (ks & 1) * 32 : ra[ks]));
    }
    // transposing read (read_tr_swz) of the rows from row0 on (a multiple of 16), columns from 32 hb on
    __device__ __forceinline__ bf16x8 tr_frag(uint32_t tile, int row0, int hb) const {
        typedef __attribute__((address_space(3))) s16x4 *lds_ptr;
        const uint32_t p = tile + rows(row0);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + ta[hb]));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + rows(8) + (HD == 128 ? ta[hb] : ta[hb] ^ 32)));
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, v);
    }
    // acc[hb] += X^T (columns hb*32.. of the tile X, reduction rows row0 ..) * frag, for all hb
    __device__ __forceinline__ void accumulate(f32x16 *acc, uint32_t tile, int row0, const bf16x8 &frag) const {
        bf16x8 a[HD / 32];
#pragma unroll
        for (int hb = 0; hb < HD / 32; ++hb) a[hb] = tr_frag(tile, row0, hb);
#pragma unroll
        for (int hb = 0; hb < HD / 32; ++hb) acc[hb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[hb], frag, acc[hb], 0, 0, 0);
    }
};

// what this wave asked for has landed, and these fragments are in their registers (here, not where a loop uses them first)
template <int N>
__device__ __forceinline__ void wave_barrier(bf16x8 (&f)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(f[i]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// the other half wave's value and the lane's own: their maximum, sum
__device__ __forceinline__ float half_max(float v) {
    const auto u = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(u[0]), __uint_as_float(u[1]));
}

__device__ __forceinline__ float half_sum(float v) {
    const auto u = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(u[0]) + __uint_as_float(u[1]);
}

__device__ __forceinline__ bf16x8 pack_frag(const f32x16 &v, int cch) {
    const int o = cch * 8;
    const uint4 u = {pack2bf(v[o + 0], v[o + 1]), pack2bf(v[o + 2], v[o + 3]), pack2bf(v[o + 4], v[o + 5]),
                     pack2bf(v[o + 6], v[o + 7])};
    return __builtin_bit_cast(bf16x8, u);
}

// Unconditional 16-byte load (callers clamp the row to the last valid one, so the loads of a fragment set
// are issued back to back instead of one branch per load; rows past the end are never stored).
__device__ __forceinline__ bf16x8 load_frag_global(const bf16_t *p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(p));
}

__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}

// lane-owned O^T / dQ^T style accumulator [HD rows][32 owned columns] -> out[owned][HD], scaled
template <int HD>
__device__ __forceinline__ void store_owned_rows(bf16_t *out_row, const f32x16 *acc, float mul, int hl) {
#pragma unroll
    for (int hb = 0; hb < HD / 32; ++hb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int j = hb * 32 + r4 * 8 + hl * 4;
            const uint2 u = {pack2bf(acc[hb][r4 * 4 + 0] * mul, acc[hb][r4 * 4 + 1] * mul),
                             pack2bf(acc[hb][r4 * 4 + 2] * mul, acc[hb][r4 * 4 + 3] * mul)};
            *reinterpret_cast<uint2 *>(out_row + j) = u;
        }
}

// The same store with the backward of the rotary embedding: the pair (j, j + HD/2) of the row is rotated by minus
// the row's angle; cs / sn point at the row's HD/2 table entries.
template <int HD>
__device__ __forceinline__ void store_owned_rows_unrotated(bf16_t *out_row, const f32x16 *acc, float mul, int hl,
                                                           const float *cs, const float *sn) {
    constexpr int HB2 = HD / 64;
#pragma unroll
    for (int hb = 0; hb < HB2; ++hb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int j = hb * 32 + r4 * 8 + hl * 4;
            const float4 c4 = *reinterpret_cast<const float4 *>(cs + j), s4 = *reinterpret_cast<const float4 *>(sn + j);
            const float c[4] = {c4.x, c4.y, c4.z, c4.w}, sv[4] = {s4.x, s4.y, s4.z, s4.w};
            float xa[4], xb[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float ya = acc[hb][r4 * 4 + e] * mul, yb = acc[hb + HB2][r4 * 4 + e] * mul;
                xa[e] = ya * c[e] + yb * sv[e];
                xb[e] = yb * c[e] - ya * sv[e];
            }
            const uint2 ua = {pack2bf(xa[0], xa[1]), pack2bf(xa[2], xa[3])};
            const uint2 ub = {pack2bf(xb[0], xb[1]), pack2bf(xb[2], xb[3])};
            *reinterpret_cast<uint2 *>(out_row + j) = ua;
            *reinterpret_cast<uint2 *>(out_row + j + HD / 2) = ub;
        }
}

// Results leave through LDS: stored from the accumulator layout (a lane owns a row) one store instruction would
// touch 64 rows with 8 bytes each.  Every wave writes its 32 x HD block into a private LDS region (free after the
// main loop's last barrier) with the two functions above and copies it out row-wise, 16 bytes per lane, whole lines.
// Falls back to the direct stores when the destination rows are not 16-byte aligned.
template <int HD>
__device__ __forceinline__ bf16_t *out_region(bf16_t *smem, int wave) { return smem + wave * 32 * (HD + 8); }

template <int HD>
__device__ __forceinline__ void flush_owned_rows(bf16_t *out_row0, int64_t ld, const bf16_t *region, int lane, int n_valid) {
    constexpr int LPR = HD / 8, RPI = 64 / LPR;
    const int lr = lane / LPR, lc = (lane % LPR) * 8;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int it = 0; it < 32 / RPI; ++it) {
        const int r = it * RPI + lr;
        if (r < n_valid)
            *reinterpret_cast<uint4 *>(out_row0 + r * ld + lc) = *reinterpret_cast<const uint4 *>(region + r * (HD + 8) + lc);
    }
}

// out_row0: row of the wave's first query / key; cs, sn: rotary tables at that row, or NULL
template <int HD>
__device__ __forceinline__ void write_owned_rows(bf16_t *out_row0, int64_t ld, const f32x16 *acc, float mul, int l32, int hl,
                                                 int n_valid, const float *cs, const float *sn, bf16_t *region) {
    const bool wide = !(ld & 7) && !((uintptr_t)out_row0 & 15);
    bf16_t *dst = wide ? region + l32 * (HD + 8) : out_row0 + l32 * ld;
    if (wide || l32 < n_valid) {
        const int tr = min(l32, n_valid - 1);  // rows past the end are never stored; keep their table reads in range
        if (cs) store_owned_rows_unrotated<HD>(dst, acc, mul, hl, cs + tr * (HD / 2), sn + tr * (HD / 2));
        else store_owned_rows<HD>(dst, acc, mul, hl);
    }
    if (wide) flush_owned_rows<HD>(out_row0, ld, region, hl * 32 + l32, n_valid);
}

// Workgroup -> (batch, KV head, item) mapping shared by the three kernels.  Consecutive workgroup ids are
// dealt round-robin to the 8 XCDs; all workgroups that read the same K/V (or Q/dO) stream are given ids
// congruent modulo 8 and adjacent in dispatch order, so they run together on one XCD and the stream is
// fetched into that XCD's L2 once.  per_set = workgroups per (batch, KV head); returns false for the
// padding workgroups of the last, partial round.
// A number of sets that is no multiple of 8 would leave XCDs idle (one set: seven of the eight), so each set is then cut into
// 2, 4 or 8 parts on different XCDs, every part an even share of light and heavy blocks: 8192 tokens, 4 query heads, 1 KV
// head of 128: forward 512 -> 213 us, dQ 708 -> 287.  Up to 7 % of idle XCD time a set stays whole (sharing one L2).
constexpr int kXcds = 8;
inline int set_parts(int n_sets) {
    int p = 1;
    while (p < kXcds && (n_sets * p + kXcds - 1) / kXcds * kXcds * 100 > n_sets * p * 107) p *= 2;
    return p;
}
// An XCD hands its workgroups to its four shader engines (8 compute units each) in turn and in order.  Up to three workgroups per
// compute unit (kByRank for an XCD's 32) the order is by rank: the heaviest block of every set, then the next one of every
// set.  With set after set an engine can get nothing but heavy blocks, and two rounds of them where one and a light block would
// do.  head_dim 128, set after set -> by rank, us: 1 x 2048, 18 heads in blocks of 128 queries (36 workgroups per XCD) forward 84.9 -> 45.5;
// 1 x 1536, 64 heads in blocks of 256 (48) 79.3 -> 52.0; 1 x 4096, 9 heads, backward in blocks of 128 472 -> 251.  Beyond that set
// after set, so that those who run together share an L2's worth of keys.  copies: blocks of one rank in a set.
constexpr int kByRank = 96;
struct BlockMap {   // worked out on the host: a workgroup of a short sequence lives for a few microseconds
    int n_sets, per_set, n_parts, per_part, log_parts;
    bool by_rank;
};
inline BlockMap block_map(int per_set, int n_sets, int copies) {
    const int p = set_parts(n_sets);
    BlockMap m = {n_sets, per_set, (n_sets * p + kXcds - 1) / kXcds, (per_set + p - 1) / p, __builtin_ctz(p), false};
    m.by_rank = (int64_t)m.n_parts * m.per_part <= kByRank && m.n_parts * copies > 1;
    return m;
}
__device__ __forceinline__ bool decode_block(const BlockMap &m, uint32_t id, int *set, int *inner) {
    const int xcd = id % kXcds, slot = id / kXcds, by = m.by_rank ? m.n_parts : m.per_part, quot = slot / by, rest = slot - quot * by;
    const int i = m.by_rank ? quot : rest, part_id = (m.by_rank ? rest : quot) * kXcds + xcd, p = 1 << m.log_parts, part = part_id & (p - 1);
    *set = part_id >> m.log_parts;
    *inner = i * p + (i & 1 ? p - 1 - part : part);
    return *set < m.n_sets && *inner < m.per_set;
}
// Division of small numbers by a number known on the host: exact while dividend times divisor stay below 2^32.
struct Div {
    uint32_t d, magic;
};
inline Div make_div(int d) { return {(uint32_t)d, d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d)}; }
__device__ __forceinline__ int quot(int x, Div v) { return v.d == 1 ? x : (int)__umulhi((uint32_t)x, v.magic); }
// One workgroup per compute unit works through a list of blocks (chain kernels): the blocks of an XCD, the parts (BlockMap) by groups
// of `group` and within a group by rank (the heaviest of every part, then the next), are dealt to its workers back and forth
// (0 .. 31, 31 .. 0, ...), so that a worker's heavy block is followed by a light one.
constexpr int kWorkers = 32;
struct ChainMap {
    int n_sets, per_set, log_parts, n_parts, n_slots, n_workers;
    Div group_slots, group_size, last_size, Hkv, G;   // slots and parts of a group, parts of the last one
    int n_blocks;
};
struct Block {
    int b, hk, h, qb;
};
// k-th entry of this workgroup's list; false: padding (nothing to do), k >= rounds: the end
__device__ __forceinline__ bool chain_block(const ChainMap &c, int k, Block *out) {
    const int xcd = blockIdx.x % kXcds, w = blockIdx.x / kXcds, slot = k * c.n_workers + (k & 1 ? c.n_workers - 1 - w : w);
    if (slot >= c.n_slots) return false;
    const int g = quot(slot, c.group_slots), rest = slot - g * (int)c.group_slots.d;
    const Div size = (g + 1) * (int)c.group_size.d <= c.n_parts ? c.group_size : c.last_size;
    const int i = quot(rest, size), part_id = (g * (int)c.group_size.d + rest - i * (int)size.d) * kXcds + xcd;
    const int p = 1 << c.log_parts, part = part_id & (p - 1), set = part_id >> c.log_parts, inner = i * p + (i & 1 ? p - 1 - part : part);
    if (set >= c.n_sets || inner >= c.per_set) return false;
    out->b = quot(set, c.Hkv);
    out->hk = set - out->b * (int)c.Hkv.d;
    const int rank = quot(inner, c.G);
    out->h = out->hk * (int)c.G.d + inner - rank * (int)c.G.d;
    out->qb = c.n_blocks - 1 - rank;
    return true;
}
struct BlockList {
    int k = 0;
    __device__ __forceinline__ bool next(const ChainMap &c, Block *out) {
        const int rounds = (c.n_slots + c.n_workers - 1) / c.n_workers;
        while (k < rounds)
            if (chain_block(c, k++, out)) return true;
        return false;
    }
};
// Causal work falls off linearly with the block index, and the workgroups of an XCD are handed to its shader
// engines round-robin in dispatch order: with the plain order "heaviest first" one engine would always get the
// heavier blocks of every set (measured: 15 us of idle time per block on the other engines' CUs at T = 4096).
// Rows of 8 consecutive positions therefore alternate direction (15..8, 0..7, ...): every residue class of the
// position modulo 8, 4 and 2 then carries the same amount of work.  i in [0, n) -> a permutation of [0, n).
__device__ __forceinline__ int snake8(int i, int n) {
    const int row = i >> 3;
    // long sequences: the classes differ by less than a percent, and the plain order keeps neighbouring blocks
    // (shared keys) together, which measured 1 % faster at 128k
    if (n > 128 || !(row & 1) || row * 8 + 7 >= n) return i;
    return row * 8 + 7 - (i & 7);
}
inline unsigned grid_blocks(const BlockMap &m) { return (unsigned)(m.n_parts * kXcds) * (unsigned)m.per_part; }

// ------------------------------------------------------------------ forward
// grid (q blocks of 32*QW rows, heaviest first; Hq; B); wave w owns 32 queries.  K and V tiles of 64
// keys go through a double-buffered LDS stage, one barrier per tile.  KW = 2: two sets of QW waves share the
// queries, one per 32-key half of every tile, and are merged through LDS at the end: half the walk per tile for problems whose
// few blocks would otherwise walk their keys while the chip idles (split_keys).  A 32-key half is either wholly
// visible to a wave's 32 queries, or the diagonal one (every query sees at least its first key), or skipped.
// One tile of 64 keys (NR = 2) or one of its halves (NR = 1, keys key0 .. + 31 of it): scores of the wave's 32 queries, their softmax, O.
// kv0: the tile's first key; q0: the wave's first query, qm: the lane's.
template <int HD, int NR>
__device__ __forceinline__ void fwd_tile(f32x16 (&oacc)[HD / 32], float &m, float &lsum, const bf16x8 (&qf)[HD / 16], const char *Ks, const char *Vs,
                                         uint32_t roff, uint32_t toff, int key0, int kv0, int q0, int qm, int hl, float c, float tau) {
    // S^T = K Q^T for the wave's 32-key row blocks: fragments are read in batches of 4 k-steps ahead of
    // the MFMAs, and the independent accumulation chains are interleaved
    f32x16 sacc[NR];
#pragma unroll
    for (int rb = 0; rb < NR; ++rb) sacc[rb] = zero16();
#pragma unroll
    for (int half = 0; half < HD / 64; ++half) {
        bf16x8 kk[NR][4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int rb = 0; rb < NR; ++rb)
                kk[rb][j] = *reinterpret_cast<const bf16x8 *>(Ks + (roff ^ ((half * 4 + j) * 32)) + (key0 + rb * 32) * (2 * HD));
        __builtin_amdgcn_sched_barrier(0);  // keep the batch of reads ahead of the MFMAs
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int rb = 0; rb < NR; ++rb)
                sacc[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[rb][j], qf[half * 4 + j], sacc[rb], 0, 0, 0);
    }
    // V^T fragments of the first two 16-key chunks are requested now, so that their LDS latency is
    // covered by the softmax arithmetic below; the other two chunks follow behind the first MFMAs
    bf16x8 va[2][HD / 32];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch)
#pragma unroll
        for (int hb = 0; hb < HD / 32; ++hb) va[ch][hb] = read_tr_swz<HD>(Vs, toff, key0 + ch * 16, hb);
    __builtin_amdgcn_sched_barrier(0);
    // Softmax on the raw scores: the scale is folded into the exponent's multiply-add, the running
    // maximum m is only moved when some query of the wave saw a score more than kLazyMax above it
    // (P then stays below 2^kLazyMax * ... which bf16 and the fp32 sums hold without loss; the final
    // O / lsum and lse do not depend on which maximum was used), so the accumulator rescale is rare.
    if (kv0 + key0 + NR * 32 - 1 > q0) {  // the keys touch the diagonal: mask those after the query
#pragma unroll
        for (int rb = 0; rb < NR; ++rb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kv = kv0 + key0 + rb * 32 + (r >> 2) * 8 + hl * 4 + (r & 3);
                sacc[rb][r] = kv > qm ? -INFINITY : sacc[rb][r];
            }
    }
    float mx = fmaxf(sacc[0][0], sacc[NR - 1][0]);
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(fmaxf(mx, sacc[0][r]), sacc[NR - 1][r]);  // v_max3_f32
    mx = half_max(mx);
    // m = -inf before the first tile: the comparison is then true (every query sees key kv0)
    if (__builtin_amdgcn_ballot_w64(mx > m + tau) != 0) {
        const float m_new = fmaxf(m, mx);
        // (queries that have seen nothing but -inf come along with the others: there is nothing to rescale yet, and
        // -inf - -inf would make a NaN of it)
        const float alpha = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f((m - m_new) * c);
        lsum *= alpha;
#pragma unroll
        for (int hb = 0; hb < HD / 32; ++hb)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[hb][r] *= alpha;
        m = m_new;
    }
    // (a query that has seen nothing but -inf so far: its P is zero)
    const float negmc = m == -INFINITY ? 0.f : -m * c;
    float ps = 0.f;
#pragma unroll
    for (int rb = 0; rb < NR; ++rb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[rb][r], c, negmc));
            sacc[rb][r] = pv;
            ps += pv;
        }
    lsum += ps;
    // O^T += V^T P^T
#pragma unroll
    for (int ch = 0; ch < 2 * NR; ++ch) {
        const bf16x8 pf = pack_frag(sacc[ch >> 1], ch & 1);
#pragma unroll
        for (int hb = 0; hb < HD / 32; ++hb)
            oacc[hb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[ch & 1][hb], pf, oacc[hb], 0, 0, 0);
        if (ch + 2 < 2 * NR) {
#pragma unroll
            for (int hb = 0; hb < HD / 32; ++hb) va[ch & 1][hb] = read_tr_swz<HD>(Vs, toff, (ch + 2) * 16, hb);
        }
    }
}

// rows of a tile that n sets of waves share, 32 of them each (a lone set takes both halves of 64)
__host__ __device__ constexpr int walk_rows(int n) { return std::max(64, 32 * n); }
// (With four waves, head_dim 128 in blocks of 32, the compiler is told of 256 registers all the same, two waves to a SIMD: given 512 it keeps accumulators
// in the other half of the register file and moves what the softmax reads back and forth.  us, forward: 1 x 1032, 4 heads on 1 14.6 -> 12.7;
// 2 x 1440, 4 on 2 19.8 -> 17.9; dQ, which has the same: 2 x 88, 20 on 4 9.0 -> 8.2, 2 x 1440, 4 on 2 24.4 -> 23.9.)
template <int HD, int QW, int KW, bool FAR>
__global__ __launch_bounds__(64 * QW * KW, 2) void flash_fwd_kernel(AttnArgs a, BlockMap map) {
    constexpr int BQ = 32 * QW, TK = walk_rows(KW), NR = TK / 32 / KW;
    constexpr uint32_t TILE = TK * HD * 2, STAGE = 2 * TILE;   // bytes; a stage is K, V
    extern __shared__ __attribute__((aligned(256))) bf16_t smem[];

    const int T = a.T, G = a.Hq / a.Hkv, nqb = (T + BQ - 1) / BQ;
    int set, inner;
    if (!decode_block(map, blockIdx.x, &set, &inner)) return;
    const int b = set / a.Hkv, hk = set % a.Hkv, h = hk * G + (map.by_rank ? inner % G : inner / nqb);
    const int qb = nqb - 1 - (map.by_rank ? inner / G : snake8(inner % nqb, nqb));  // heaviest query blocks first (in alternating rows of 8)
    const int lane = threadIdx.x & 63, wave = wave_index(), l32 = lane & 31, hl = lane >> 5;
    const uint32_t roff = row_off<HD>(l32, hl), toff = tr_off_swz<HD>(lane);
    const int qw = wave % QW, kw = wave / QW;
    const int q0 = qb * BQ + qw * 32, q = q0 + l32;
    const bool qok = q < T;
    const int qm = qok ? q : T - 1;  // padded queries behave like the last row; never stored

    const bf16_t *kbase = a.k + (int64_t)b * T * a.ldk + (int64_t)hk * HD;
    const bf16_t *vbase = a.v + (int64_t)b * T * a.ldv + (int64_t)hk * HD;
    const int kv_end = min(T, qb * BQ + BQ);
    const int ntiles = (kv_end + TK - 1) / TK;
    DirectTile<TK, HD, QW * KW, FAR> dk, dv;
    dk.init(smem, a.ldk, lane, wave);
    dv.init(smem, a.ldv, lane, wave);
    dk.load(0, kbase, a.ldk, 0, T);
    dv.load(TILE, vbase, a.ldv, 0, T);

    bf16x8 qf[HD / 16];
    {
        const bf16_t *qp = a.q + ((int64_t)b * T + qm) * a.ldq + (int64_t)h * HD + hl * 8;
#pragma unroll
        for (int ks = 0; ks < HD / 16; ++ks) qf[ks] = load_frag_global(qp + ks * 16);
    }
    f32x16 oacc[HD / 32];
#pragma unroll
    for (int hb = 0; hb < HD / 32; ++hb) oacc[hb] = zero16();
    float m = -INFINITY, lsum = 0.f;  // m: running maximum of the raw (unscaled) scores
    const float c = a.scale * kLog2e, tau = kLazyMax / c;
    const int key0 = KW > 1 ? kw * 32 : 0;  // first key of this wave inside a tile
    tile_barrier();

    const auto step = [&](int kt, uint32_t stage) {
        const int kv0 = kt * TK;
        if (kt + 1 < ntiles) {
            dk.load(STAGE - stage, kbase, a.ldk, kv0 + TK, T);
            dv.load(STAGE - stage + TILE, vbase, a.ldv, kv0 + TK, T);
        }
        if (kv0 + key0 <= q0 + 31 && q0 < T) {  // otherwise the wave's keys lie after every one of its queries, or it has none
            const char *Ks = reinterpret_cast<const char *>(smem) + stage;
            fwd_tile<HD, NR>(oacc, m, lsum, qf, Ks, Ks + TILE, roff, toff, key0, kv0, q0, qm, hl, c, tau);
        }
        tile_barrier();
    };
    for (int kt = 0; kt < ntiles; kt += 2) {   // by twos: the LDS addresses are then constants
        step(kt, 0);
        if (kt + 1 < ntiles) step(kt + 1, STAGE);
    }
    lsum += __shfl_xor(lsum, 32, 64);
    if constexpr (KW == 2) {
        constexpr int NV = HD / 32 * 16;
        float *red = reinterpret_cast<float *>(smem) + qw * ((NV + 2) * 64) + lane;
        if (kw == 1) {
#pragma unroll
            for (int i = 0; i < NV; ++i) red[i * 64] = oacc[i / 16][i % 16];
            red[NV * 64] = m;   // -inf where this half saw no key: its weight below is zero
            red[(NV + 1) * 64] = lsum;
        }
        __syncthreads();
        if (kw == 0) {
            const float m1 = red[NV * 64], mn = fmaxf(m, m1);
            const float w0 = __builtin_amdgcn_exp2f((m - mn) * c), w1 = __builtin_amdgcn_exp2f((m1 - mn) * c);
            lsum = lsum * w0 + red[(NV + 1) * 64] * w1;
            m = mn;
#pragma unroll
            for (int i = 0; i < NV; ++i) oacc[i / 16][i % 16] = oacc[i / 16][i % 16] * w0 + red[i * 64] * w1;
        }
        __syncthreads();
        if (kw == 1) return;
    }
    if constexpr (KW > 2) {   // as above, but all waves add: each a share of the columns of its QW neighbours' 32 queries
        constexpr int QUADS = HD / 32 * 4;
        f32x4 *sums = reinterpret_cast<f32x4 *>(smem);
        float *stat = reinterpret_cast<float *>(smem) + QW * KW * (QUADS * 256);
#pragma unroll
        for (int i = 0; i < QUADS; ++i)
            sums[(wave * QUADS + i) * 64 + lane] = f32x4{oacc[i >> 2][(i & 3) * 4], oacc[i >> 2][(i & 3) * 4 + 1], oacc[i >> 2][(i & 3) * 4 + 2], oacc[i >> 2][(i & 3) * 4 + 3]};
        stat[wave * 128 + lane] = m;   // -inf where this share saw no key: its weight below is zero
        stat[wave * 128 + 64 + lane] = lsum;
        __syncthreads();
        float w[KW], mn = -INFINITY, sum = 0.f;
#pragma unroll
        for (int i = 0; i < KW; ++i) {
            w[i] = stat[(i * QW + qw) * 128 + lane];
            mn = fmaxf(mn, w[i]);
        }
#pragma unroll
        for (int i = 0; i < KW; ++i) {
            w[i] = __builtin_amdgcn_exp2f((w[i] - mn) * c);
            sum += stat[(i * QW + qw) * 128 + 64 + lane] * w[i];
        }
        if (!qok) return;
        bf16_t *out = a.o + ((int64_t)b * T + q) * a.ldo + (int64_t)h * HD;
        const float mul = 1.0f / sum;
        for (int p = kw; p < QUADS; p += KW) {
            f32x4 x = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < KW; ++i) x += sums[((i * QW + qw) * QUADS + p) * 64 + lane] * w[i];
            *reinterpret_cast<uint2 *>(out + (p >> 2) * 32 + (p & 3) * 8 + hl * 4) = uint2{pack2bf(x[0] * mul, x[1] * mul), pack2bf(x[2] * mul, x[3] * mul)};
        }
        if (kw == 0 && hl == 0) a.lse[((int64_t)b * a.Hq + h) * T + q] = (mn * c + __builtin_amdgcn_logf(sum)) * kLn2;
        return;
    }
    if (q0 < T)
        write_owned_rows<HD>(a.o + ((int64_t)b * T + q0) * a.ldo + (int64_t)h * HD, a.ldo, oacc, 1.0f / lsum, l32, hl,
                             min(32, T - q0), nullptr, nullptr, out_region<HD>(smem, qw));
    if (qok && hl == 0) a.lse[((int64_t)b * a.Hq + h) * T + q] = (m * c + __builtin_amdgcn_logf(lsum)) * kLn2;
}

// The wave's 32 x HD results through 64 COLS bytes of its own, COLS columns at a time (see write_owned_rows).
template <int HD, int COLS>
__device__ __forceinline__ void write_rows_by_parts(bf16_t *out_row0, int64_t ld, const f32x16 *acc, float mul, int l32, int hl, int n_valid, char *region) {
    if ((ld & 7) || ((uintptr_t)out_row0 & 15)) {
        if (l32 < n_valid) store_owned_rows<HD>(out_row0 + l32 * ld, acc, mul, hl);
        return;
    }
    constexpr int CH = COLS / 8, RPI = 64 / CH;   // chunks of 16 bytes per row, rows per store
    const int lane = hl * 32 + l32, lr = lane / CH, lc = lane % CH;
#pragma unroll
    for (int part = 0; part < HD / COLS; ++part) {
#pragma unroll
        for (int h = 0; h < COLS / 32; ++h)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const f32x16 &v = acc[part * (COLS / 32) + h];
                const uint2 u = {pack2bf(v[r4 * 4 + 0] * mul, v[r4 * 4 + 1] * mul), pack2bf(v[r4 * 4 + 2] * mul, v[r4 * 4 + 3] * mul)};
                *reinterpret_cast<uint2 *>(region + l32 * (2 * COLS) + (((h * 4 + r4) ^ (l32 & (CH - 1))) << 4) + hl * 8) = u;
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int r = it * RPI + lr;
            const uint4 u = *reinterpret_cast<const uint4 *>(region + r * (2 * COLS) + ((lc ^ (r & (CH - 1))) << 4));
            if (r < n_valid) *reinterpret_cast<uint4 *>(out_row0 + r * ld + part * COLS + lc * 8) = u;
        }
    }
}
// The backward of the rotary embedding on the lane's row (see store_owned_rows_unrotated), times mul
template <int HD>
__device__ __forceinline__ void rotate_back(f32x16 *acc, float mul, int hl, const float *cs, const float *sn) {
#pragma unroll
    for (int hb = 0; hb < HD / 64; ++hb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const int j = hb * 32 + r4 * 8 + hl * 4;
            const float4 c4 = *reinterpret_cast<const float4 *>(cs + j), s4 = *reinterpret_cast<const float4 *>(sn + j);
            const float c[4] = {c4.x, c4.y, c4.z, c4.w}, sv[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float ya = acc[hb][r4 * 4 + e] * mul, yb = acc[hb + HD / 64][r4 * 4 + e] * mul;
                acc[hb][r4 * 4 + e] = ya * c[e] + yb * sv[e];
                acc[hb + HD / 64][r4 * 4 + e] = yb * c[e] - ya * sv[e];
            }
        }
}

// The same forward in blocks of 256 queries with one workgroup per compute unit that goes through a list of them.  A block of its own
// workgroup spends 4-5 us on its start (queries, first tile) and its results, next to 1.9 us per tile, and workgroups that are handed out in
// order leave compute units idle; here the first tile and the queries of the next block are requested during the present one, a wave
// writes its results as soon as its own last tile is done, while the waves with later queries still work on theirs, and the lists
// share the work evenly.  us, a workgroup per block (with tiles through registers) -> now: 4 x 4096, 32 heads 650 -> 554 (995 TFLOP/s);
// 8 x 2048, 16 heads 212 -> 153; 8 x 1024, 32 heads 141 -> 98; 1 x 32768, 40 heads on 8 10 927 -> 9869 (6 % of it by loads that write LDS).
// head_dim 64, blocks of 128 -> lists: 8 x 2048, 16 heads 129 -> 94 (backward, lists there too, 406 -> 282); 8 x 1024, 32 heads 70 -> 53 (245 -> 170).
// What bounds it now: matrix pipes busy for 46 % of the cycles at 1.85 GHz (counters, 16 x 4096, 32 heads), 4.9 vector instructions for each of the matrix
// pipe's, which share its issue port, and the power limit.
// LDS: two stages of K and V | the wave's queries of the next block | the wave's results on their way out
template <int HD>
__global__ __launch_bounds__(512) void flash_fwd_chain_kernel(AttnArgs a, ChainMap map) {
    constexpr int BQ = 256;
    constexpr uint32_t TILE = 64 * HD * 2, STAGE = 2 * TILE, Q_OFF = 2 * STAGE, O_OFF = Q_OFF + BQ * HD * 2;
    extern __shared__ __attribute__((aligned(256))) bf16_t smem[];
    char *lds = reinterpret_cast<char *>(smem);
    const int T = a.T;
    const int lane = threadIdx.x & 63, wave = wave_index(), l32 = lane & 31, hl = lane >> 5;
    const uint32_t roff = row_off<HD>(l32, hl), toff = tr_off_swz<HD>(lane);
    const float c = a.scale * kLog2e, tau = kLazyMax / c;

    DirectTile<64, HD, 8, false> dk, dv;
    DirectTile<32, HD, 1, false> dq;   // a wave fetches its own queries
    dk.init(smem, a.ldk, lane, wave);
    dv.init(smem, a.ldv, lane, wave);
    dq.init(smem, a.ldq, lane, 0);
    const uint32_t q_lds = Q_OFF + wave * (32 * HD * 2);

    BlockList list;
    Block cur, nxt;
    const auto request_tile = [&](const Block &blk, int kt, uint32_t stage) {
        dk.load(stage, a.k + (int64_t)blk.b * T * a.ldk + (int64_t)blk.hk * HD, a.ldk, kt * 64, T);
        dv.load(stage + TILE, a.v + (int64_t)blk.b * T * a.ldv + (int64_t)blk.hk * HD, a.ldv, kt * 64, T);
    };
    const auto request_queries = [&](const Block &blk) {
        dq.load(q_lds, a.q + (int64_t)blk.b * T * a.ldq + (int64_t)blk.h * HD, a.ldq, blk.qb * BQ + wave * 32, T);
    };
    if (!list.next(map, &cur)) return;
    request_queries(cur);
    request_tile(cur, 0, 0);
    tile_barrier();
    while (true) {
        bf16x8 qf[HD / 16];
#pragma unroll
        for (int ks = 0; ks < HD / 16; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(lds + q_lds + (roff ^ (ks * 32)));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const bool more = list.next(map, &nxt);
        if (more) request_queries(nxt);
        const int q0 = cur.qb * BQ + wave * 32, q = q0 + l32, qm = min(q, T - 1);  // padded queries behave like the last row; never stored
        const int ntiles = (min(T, cur.qb * BQ + BQ) + 63) / 64, last = q0 < T ? min(ntiles, (q0 + 31) / 64 + 1) - 1 : -1;   // (no tile for queries past the end)
        f32x16 oacc[HD / 32];
#pragma unroll
        for (int hb = 0; hb < HD / 32; ++hb) oacc[hb] = zero16();
        float m = -INFINITY, lsum = 0.f;
        const auto request_after = [&](int kt, uint32_t stage) {
            if (kt + 1 < ntiles) request_tile(cur, kt + 1, STAGE - stage);
            else if (more && (kt & 1)) request_tile(nxt, 0, STAGE - stage);
        };
        const auto step = [&](int kt, uint32_t stage) {
            request_after(kt, stage);
            if (kt <= last) fwd_tile<HD, 2>(oacc, m, lsum, qf, lds + stage, lds + stage + TILE, roff, toff, 0, kt * 64, q0, qm, hl, c, tau);
            tile_barrier();
        };
        int kt = 0;
        for (; kt <= last; kt += 2) {   // by twos: the LDS addresses are then constants, and every block starts in stage 0
            step(kt, 0);
            step(kt + 1, STAGE);
        }
        const float sum = half_sum(lsum);
        if (q0 < T)
            write_rows_by_parts<HD, 64>(a.o + ((int64_t)cur.b * T + q0) * a.ldo + (int64_t)cur.h * HD, a.ldo, oacc, 1.0f / sum, l32, hl,
                                        min(32, T - q0), lds + O_OFF + wave * 4096);
        if (q < T && hl == 0) a.lse[((int64_t)cur.b * a.Hq + cur.h) * T + q] = (m * c + __builtin_amdgcn_logf(sum)) * kLn2;
        for (; kt < ntiles; kt += 2) {   // the other waves' tiles
            request_after(kt, 0);
            tile_barrier();
            request_after(kt + 1, STAGE);
            tile_barrier();
        }
        if (!more) break;
        cur = nxt;
    }
}

// ------------------------------------------------------------------ backward: dQ
// Same ownership as the forward: a lane owns one query, loops over key tiles <= q.
// KW = 2 splits the tiles' keys over two sets of waves as in the forward; their sums are added at the end.

// dQ is the first kernel of the backward: it has the output gradients of its queries at hand, so it also works out delta = rowsum(dO * O),
// which is stored for dK/dV (a pass of its own read dO once more.  us, forward and backward, with -> without it: 3 x 520, 8 heads of 64 on 2 40.6 -> 38.6;
// 4 x 4096, 32 heads 2518 -> 2502; 1 x 32768, 40 heads on 8 43 830 -> 43 740).
// (A product of two bf16 is exact in fp32, so a pair of terms is rounded once.  The two-element dot product instruction adds the terms one by one instead:
// where neighbouring terms cancel it loses what was there before.)
__device__ __forceinline__ float dot8(const bf16x8 &x, const bf16x8 &y) {
    const u32x4 a = __builtin_bit_cast(u32x4, x), b = __builtin_bit_cast(u32x4, y);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) s += bflo(a[i]) * bflo(b[i]) + bfhi(a[i]) * bfhi(b[i]);
    return s;
}
template <int HD>
__device__ __forceinline__ float row_delta(const bf16x8 (&dof)[HD / 16], const bf16x8 (&of)[HD / 16]) {
    float s[2] = {0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < HD / 16; ++ks) s[ks & 1] += dot8(dof[ks], of[ks]);
    return half_sum(s[0] + s[1]);
}

// the keys 32 rb .. + 31 (rb0 <= rb < rb0 + NR) of the tile that starts at key kv0
template <int HD, int NR>
__device__ __forceinline__ void dq_tile(f32x16 (&dqacc)[HD / 32], const bf16x8 (&qf)[HD / 16], const bf16x8 (&dof)[HD / 16], uint32_t Ks, uint32_t Vs,
                                        const BwdTile<HD> &t, int rb0, int kv0, int q0, int qm, int hl, float c, float lse2, float dlt) {
    const bool diag = kv0 + (NR == 1 ? rb0 * 32 + 31 : 63) > q0;
#pragma unroll
    for (int u = 0; u < NR; ++u) {
        const int rb = NR == 1 ? rb0 : u;
        const uint32_t Kr = Ks + BwdTile<HD>::rows(rb * 32), Vr = Vs + BwdTile<HD>::rows(rb * 32);
        f32x16 sacc = zero16(), dpacc = zero16();
#pragma unroll
        for (int half = 0; half < HD / 64; ++half) {
            bf16x8 kk[4], vv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                kk[j] = t.row_frag(Kr, half * 4 + j);
                vv[j] = t.row_frag(Vr, half * 4 + j);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[j], qf[half * 4 + j], sacc, 0, 0, 0);
                dpacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv[j], dof[half * 4 + j], dpacc, 0, 0, 0);
            }
        }
        if (diag) {  // wave-uniform: only tiles that touch the diagonal pay for the mask
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int kv = kv0 + rb * 32 + (r >> 2) * 8 + hl * 4 + (r & 3);
                const float p = kv > qm ? 0.f : __builtin_amdgcn_exp2f(sacc[r] * c - lse2);
                sacc[r] = p * (dpacc[r] - dlt);  // dS^T
            }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                sacc[r] = __builtin_amdgcn_exp2f(sacc[r] * c - lse2) * (dpacc[r] - dlt);
        }
        // dQ^T += K^T dS^T
#pragma unroll
        for (int cch = 0; cch < 2; ++cch) t.accumulate(dqacc, Kr, cch * 16, pack_frag(sacc, cch));
    }
}

// The sums of N sets of W waves that shared a block, added up in the order of the sets and stored.  Wave w of every set owns the same 32 rows
// (a lane one of them, at out); each adds and stores a share of their columns, so all of them work on it.  cs, sn: rotary tables at the row, or NULL.
template <int HD, int W, int N>
__device__ __forceinline__ void store_summed(bf16_t *out, const f32x16 *acc, float mul, int w, int set, int lane, bool valid,
                                             const float *cs, const float *sn, char *smem) {
    constexpr int HB = HD / 32, QUADS = HB * 4, PAIRS = HD / 64 * 4;   // quads of columns of a lane; pairs of them that rotate together
    f32x4 *mine = reinterpret_cast<f32x4 *>(smem) + (set * W + w) * (QUADS * 64) + lane;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < QUADS; ++i)
        mine[i * 64] = f32x4{acc[i >> 2][(i & 3) * 4], acc[i >> 2][(i & 3) * 4 + 1], acc[i >> 2][(i & 3) * 4 + 2], acc[i >> 2][(i & 3) * 4 + 3]};
    __syncthreads();
    if (!valid) return;
    const f32x4 *first = reinterpret_cast<const f32x4 *>(smem) + w * (QUADS * 64) + lane;
    for (int p = set; p < PAIRS; p += N) {
        f32x4 x = first[p * 64], y = first[(p + PAIRS) * 64];
#pragma unroll
        for (int s = 1; s < N; ++s) {
            x += first[(s * W * QUADS + p) * 64];
            y += first[(s * W * QUADS + p + PAIRS) * 64];
        }
        const int j = (p >> 2) * 32 + (p & 3) * 8 + (lane >> 5) * 4;
        x *= mul;
        y *= mul;
        if (cs) {
            const f32x4 c = *reinterpret_cast<const f32x4 *>(cs + j), v = *reinterpret_cast<const f32x4 *>(sn + j);
            const f32x4 r = x * c + y * v;
            y = y * c - x * v;
            x = r;
        }
        *reinterpret_cast<uint2 *>(out + j) = uint2{pack2bf(x[0], x[1]), pack2bf(x[2], x[3])};
        *reinterpret_cast<uint2 *>(out + j + HD / 2) = uint2{pack2bf(y[0], y[1]), pack2bf(y[2], y[3])};
    }
}
// (a block; the kernel follows)
template <int HD, int QW, int KW, bool FAR>
__device__ __forceinline__ void dq_block(const AttnArgs &a, const BlockMap &map, uint32_t id, bf16_t *smem) {
    constexpr int BQ = 32 * QW, TK = walk_rows(KW);
    constexpr uint32_t TILE = BwdTile<HD>::rows(TK), STAGE = 2 * TILE;   // a stage is K, V

    const int T = a.T, G = a.Hq / a.Hkv, nqb = (T + BQ - 1) / BQ;
    int set, inner;
    if (!decode_block(map, id, &set, &inner)) return;
    const int b = set / a.Hkv, hk = set % a.Hkv, h = hk * G + (map.by_rank ? inner % G : inner / nqb);
    const int qb = nqb - 1 - (map.by_rank ? inner / G : snake8(inner % nqb, nqb));
    const int lane = threadIdx.x & 63, wave = wave_index(), l32 = lane & 31, hl = lane >> 5;
    BwdTile<HD> t;
    t.init(smem, lane);
    const int qw = wave % QW, kw = wave / QW;
    const int q0 = qb * BQ + qw * 32, q = q0 + l32;
    const bool qok = q < T;
    const int qm = qok ? q : T - 1;

    const bf16_t *kbase = a.k + (int64_t)b * T * a.ldk + (int64_t)hk * HD;
    const bf16_t *vbase = a.v + (int64_t)b * T * a.ldv + (int64_t)hk * HD;
    const int kv_end = min(T, qb * BQ + BQ);
    const int ntiles = (kv_end + TK - 1) / TK;
    DirectTile<TK, HD, QW * KW, FAR, BwdTile<HD>::GS> tk, tv;
    tk.init(smem, a.ldk, lane, wave);
    tv.init(smem, a.ldv, lane, wave);
    tk.load(0, kbase, a.ldk, 0, T);
    tv.load(TILE, vbase, a.ldv, 0, T);

    bf16x8 qf[HD / 16], dof[HD / 16];
    {
        const bf16_t *qp = a.q + ((int64_t)b * T + qm) * a.ldq + (int64_t)h * HD + hl * 8;
        const bf16_t *dp = a.dout + ((int64_t)b * T + qm) * a.lddo + (int64_t)h * HD + hl * 8;
#pragma unroll
        for (int ks = 0; ks < HD / 16; ++ks) {
            qf[ks] = load_frag_global(qp + ks * 16);
            dof[ks] = load_frag_global(dp + ks * 16);
        }
    }
    const int64_t stat = ((int64_t)b * a.Hq + h) * T + qm;
    const float lse2 = a.lse[stat] * kLog2e;
    float dlt;
    if (a.o) {
        bf16x8 of[HD / 16];
        const bf16_t *op = a.o + ((int64_t)b * T + qm) * a.ldo + (int64_t)h * HD + hl * 8;
#pragma unroll
        for (int ks = 0; ks < HD / 16; ++ks) of[ks] = load_frag_global(op + ks * 16);
        dlt = row_delta<HD>(dof, of);
        if (qok && kw == 0 && hl == 0) a.delta[stat] = dlt;
    } else {
        dlt = a.delta[stat];
    }
    const float c = a.scale * kLog2e;
    f32x16 dqacc[HD / 32];
#pragma unroll
    for (int hb = 0; hb < HD / 32; ++hb) dqacc[hb] = zero16();
    tile_barrier();

    const auto step = [&](int kt, uint32_t stage) {
        const int kv0 = kt * TK;
        if (kt + 1 < ntiles) {
            tk.load(STAGE - stage, kbase, a.ldk, kv0 + TK, T);
            tv.load(STAGE - stage + TILE, vbase, a.ldv, kv0 + TK, T);
        }
        if (kv0 + (KW > 1 ? kw * 32 : 0) <= q0 + 31 && q0 < T) {
            dq_tile<HD, TK / 32 / KW>(dqacc, qf, dof, stage, stage + TILE, t, kw, kv0, q0, qm, hl, c, lse2, dlt);
        }
        tile_barrier();
    };
    for (int kt = 0; kt < ntiles; kt += 2) {   // by twos: the LDS addresses are then constants
        step(kt, 0);
        if (kt + 1 < ntiles) step(kt + 1, STAGE);
    }
    if constexpr (KW == 2) {
        constexpr int NV = HD / 32 * 16;
        float *red = reinterpret_cast<float *>(smem) + qw * (NV * 64) + lane;
        if (kw == 1) {
#pragma unroll
            for (int i = 0; i < NV; ++i) red[i * 64] = dqacc[i / 16][i % 16];
        }
        __syncthreads();
        if (kw == 0) {
#pragma unroll
            for (int i = 0; i < NV; ++i) dqacc[i / 16][i % 16] += red[i * 64];
        }
        __syncthreads();
        if (kw == 1) return;
    }
    if constexpr (KW > 2) {
        store_summed<HD, QW, KW>(a.dq + ((int64_t)b * T + q) * a.lddq + (int64_t)h * HD, dqacc, a.scale, qw, kw, lane, qok,
                                 a.rope_cos ? a.rope_cos + (int64_t)qm * (HD / 2) : nullptr, a.rope_cos ? a.rope_sin + (int64_t)qm * (HD / 2) : nullptr,
                                 reinterpret_cast<char *>(smem));
        return;
    }
    if (q0 < T)
        write_owned_rows<HD>(a.dq + ((int64_t)b * T + q0) * a.lddq + (int64_t)h * HD, a.lddq, dqacc, a.scale, l32, hl,
                             min(32, T - q0), a.rope_cos ? a.rope_cos + (int64_t)q0 * (HD / 2) : nullptr,
                             a.rope_cos ? a.rope_sin + (int64_t)q0 * (HD / 2) : nullptr, out_region<HD>(smem, qw));
}
template <int HD, int QW, int KW, bool FAR>
__global__ __launch_bounds__(64 * QW * KW, 2) void flash_bwd_dq_kernel(AttnArgs a, BlockMap map) {
    extern __shared__ __attribute__((aligned(256))) bf16_t smem[];
    dq_block<HD, QW, KW, FAR>(a, map, blockIdx.x, smem);
}

// The same in blocks of 256 queries with one workgroup per compute unit that goes through a list of them (see flash_fwd_chain_kernel).  The
// queries and output gradients of the next block come straight into their registers as soon as the wave is done with the present one.
// us, backward, a workgroup per block -> lists (dK/dV too): 4 x 4096, 32 heads 1952 -> 1890; 8 x 2048, 16 heads 651 -> 547; 8 x 1024, 32 heads
// 458 -> 353; 1 x 32768, 40 heads on 8 32 890 -> 32 600.  Bound like the forward; short lists are no slower (1 x 1536, 64 heads 165.5 both).
template <int HD>
__global__ __launch_bounds__(512) void flash_bwd_dq_chain_kernel(AttnArgs a, ChainMap map) {
    constexpr int BQ = 256;
    constexpr uint32_t TILE = BwdTile<HD>::BYTES, STAGE = 2 * TILE, O_OFF = 2 * STAGE;
    extern __shared__ __attribute__((aligned(256))) bf16_t smem[];
    const int T = a.T;
    const int lane = threadIdx.x & 63, wave = wave_index(), l32 = lane & 31, hl = lane >> 5;
    BwdTile<HD> t;
    t.init(smem, lane);
    const float c = scalar(a.scale * kLog2e);
    DirectTile<64, HD, 8, false, BwdTile<HD>::GS> tk, tv;
    tk.init(smem, a.ldk, lane, wave);
    tv.init(smem, a.ldv, lane, wave);

    bf16x8 qf[HD / 16], dof[HD / 16], of[HD / 16];
    float lse;
    const auto request_tile = [&](const Block &blk, int kt, uint32_t stage) {
        tk.load(stage, a.k + (int64_t)blk.b * T * a.ldk + (int64_t)blk.hk * HD, a.ldk, kt * 64, T);
        tv.load(stage + TILE, a.v + (int64_t)blk.b * T * a.ldv + (int64_t)blk.hk * HD, a.ldv, kt * 64, T);
    };
    const auto request_queries = [&](const Block &blk) {
        const int qm = min(blk.qb * BQ + wave * 32 + l32, T - 1);
        const bf16_t *qp = a.q + ((int64_t)blk.b * T + qm) * a.ldq + (int64_t)blk.h * HD + hl * 8;
        const bf16_t *dp = a.dout + ((int64_t)blk.b * T + qm) * a.lddo + (int64_t)blk.h * HD + hl * 8;
#pragma unroll
        for (int ks = 0; ks < HD / 16; ++ks) {
            qf[ks] = load_frag_global(qp + ks * 16);
            dof[ks] = load_frag_global(dp + ks * 16);
        }
        lse = a.lse[((int64_t)blk.b * a.Hq + blk.h) * T + qm];
    };
    const auto request_outputs = [&](const Block &blk) {   // (without a condition: what may keep its value here would hold its registers through the whole block)
        const int qm = min(blk.qb * BQ + wave * 32 + l32, T - 1);
        const bf16_t *op = (a.o ? a.o : a.dout) + ((int64_t)blk.b * T + qm) * (a.o ? a.ldo : a.lddo) + (int64_t)blk.h * HD + hl * 8;
#pragma unroll
        for (int ks = 0; ks < HD / 16; ++ks) of[ks] = load_frag_global(op + ks * 16);
    };
    BlockList list;
    Block cur, nxt;
    if (!list.next(map, &cur)) return;
    request_tile(cur, 0, 0);
    request_queries(cur);
    request_outputs(cur);
    tile_barrier();
    while (true) {
        asm volatile("" : "+v"(lse));
        wave_barrier(qf);
        wave_barrier(dof);
        wave_barrier(of);
        const bool more = list.next(map, &nxt);
        const int q0 = cur.qb * BQ + wave * 32, q = q0 + l32, qm = min(q, T - 1);
        const int ntiles = (min(T, cur.qb * BQ + BQ) + 63) / 64, last = q0 < T ? min(ntiles, (q0 + 31) / 64 + 1) - 1 : -1;   // (no tile for queries past the end)
        const int64_t stat = ((int64_t)cur.b * a.Hq + cur.h) * T + qm;
        const float lse2 = lse * kLog2e;
        float delta;
        if (a.o) {
            delta = row_delta<HD>(dof, of);
            if (q < T && hl == 0) a.delta[stat] = delta;
        } else {
            delta = a.delta[stat];
        }
        f32x16 dqacc[HD / 32];
#pragma unroll
        for (int hb = 0; hb < HD / 32; ++hb) dqacc[hb] = zero16();
        const auto request_after = [&](int kt, uint32_t stage) {
            if (kt + 1 < ntiles) request_tile(cur, kt + 1, STAGE - stage);
            else if (more && (kt & 1)) request_tile(nxt, 0, STAGE - stage);
        };
        const auto step = [&](int kt, uint32_t stage) {
            request_after(kt, stage);
            if (kt <= last) dq_tile<HD, 2>(dqacc, qf, dof, stage, stage + TILE, t, 0, kt * 64, q0, qm, hl, c, lse2, delta);
            tile_barrier();
        };
        int kt = 0;
        for (; kt <= last; kt += 2) {
            step(kt, 0);
            step(kt + 1, STAGE);
        }
        if (more) request_queries(nxt);
        if (q0 < T) {
            const bool rope = a.rope_cos != nullptr;
            if (rope) rotate_back<HD>(dqacc, a.scale, hl, a.rope_cos + (int64_t)qm * (HD / 2), a.rope_sin + (int64_t)qm * (HD / 2));
            write_rows_by_parts<HD, 64>(a.dq + ((int64_t)cur.b * T + q0) * a.lddq + (int64_t)cur.h * HD, a.lddq, dqacc, rope ? 1.0f : a.scale, l32, hl,
                                        min(32, T - q0), reinterpret_cast<char *>(smem) + O_OFF + wave * 4096);
        }
        __builtin_amdgcn_sched_barrier(0);
        request_outputs(more ? nxt : cur);   // (in the place of the results)
        for (; kt < ntiles; kt += 2) {
            request_after(kt, 0);
            tile_barrier();
            request_after(kt + 1, STAGE);
            tile_barrier();
        }
        if (!more) break;
        cur = nxt;
    }
}

// ------------------------------------------------------------------ backward: dK, dV
// grid: key blocks of 256 (heaviest first = block 0) x (batch, KV head); the query heads of the group and their
// 64-query tiles >= the key block are walked as one sequence through a double-buffered LDS stage, one barrier
// per tile.  8 waves, two per SIMD: wave w owns keys w*32 .. w*32+31 of the block (a lane owns one key) and works
// through both 32-query halves of every tile: S^T = K Q^T and dP^T = V dO^T (16 MFMAs), P = exp2(S c - lse),
// dS = P (dP - delta) on the vector ALU, then dV^T += dO^T P and dK^T += Q^T dS (16 MFMAs); the other wave's MFMAs
// cover the exponentials.  The lane's K fragments live in registers, its V fragments are re-read from LDS for
// every half: with both in registers only one wave fits on a SIMD (that version, with a three-stage software
// pipeline inside the wave to make up for it, measured 25 % slower at 128k tokens).  A block of 256 keys rather
// than 128 halves the Q / dO bytes fetched and written to LDS per MFMA.
// LDS: two stages of Q, dO (first: their addresses are then constants of the instructions) | V | their lse * log2e [64], delta [64].
//
// The work of a key block is one serial walk over G T / 64 tiles, so a short or narrow problem leaves most of the chip
// idle while its few blocks walk.  KW, QW: KW waves own 32 keys each (blocks of 32 KW keys); with QW = 2 two such sets
// share a block, one per 32-query half of every tile, and the second set's sums are added to the first's through
// LDS at the end (fixed order).  (8, 1) above is the cheapest per tile, (4, 2) and (2, 2) have shorter walks: see
// choose_dkdv.

// the queries 32 rb .. + 31 (rb0 <= rb < rb0 + NR) of the tile that starts at query q0t; kv0w: the wave's first key, kv: the lane's;
// stats: lse * log2e [TQ], delta [TQ] from the lane half's first query on; Vw: the wave's rows of V
// (VREG: vf instead)
template <int HD, int NR, bool TIGHT, int TQ = 64, bool VREG = false>
__device__ __forceinline__ void dkdv_tile(f32x16 (&dvacc)[HD / 32], f32x16 (&dkacc)[HD / 32], const bf16x8 (&kf)[HD / 16], uint32_t Qs, uint32_t dOs,
                                          uint32_t stats, uint32_t Vw, const BwdTile<HD> &t, int rb0, int q0t, int kv0w, int kv, int hl, float c,
                                          const bf16x8 *vf = nullptr) {
    typedef __attribute__((address_space(3))) const f32x4 *lds_f4;
#pragma unroll
    for (int u = 0; u < NR; ++u) {
        const int rb = NR == 1 ? rb0 : u, q0u = q0t + rb * 32;
        if (q0u + 31 < kv0w) continue;  // wave-uniform: no query of the half sees a key of the wave
        f32x16 s_ = zero16(), p_ = zero16();
        const uint32_t qr = Qs + BwdTile<HD>::rows(rb * 32), dor = dOs + BwdTile<HD>::rows(rb * 32);
#pragma unroll
        for (int half = 0; half < HD / 64; ++half) {
            bf16x8 qq[4], dd[4], vv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) qq[i] = t.row_frag(qr, half * 4 + i);
            // TIGHT: in two batches, for with all fragments on their way the registers do not suffice, and values that are brought back
            // from scratch memory wait for the tile loads in front of them (4 x 4096, 32 heads: backward 2336 us, without 1996)
            if constexpr (TIGHT) {
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 4; ++i) s_ = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qq[i], kf[half * 4 + i], s_, 0, 0, 0);
                asm volatile("" : "+v"(s_) : : "memory");
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                dd[i] = t.row_frag(dor, half * 4 + i);
                vv[i] = VREG ? vf[half * 4 + i] : t.row_frag(Vw, half * 4 + i);
            }
            if constexpr (!TIGHT) {
#pragma unroll
                for (int i = 0; i < 4; ++i) s_ = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qq[i], kf[half * 4 + i], s_, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) p_ = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dd[i], vv[i], p_, 0, 0, 0);
            if constexpr (TIGHT) asm volatile("" : "+v"(p_) : : "memory");
        }
        // P = exp2(S c - lse), dS = P (dP - delta); element r of the lane belongs to query
        // q0u + (r >> 2) * 8 + hl * 4 + (r & 3), visible to the lane's key only if kv <= query
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const f32x4 lv = *(lds_f4)(stats + (rb * 32 + r4 * 8) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) s_[r4 * 4 + e] = __builtin_amdgcn_exp2f(s_[r4 * 4 + e] * c - lv[e]);
        }
        if (q0u < kv0w + 31) {   // (scalar: only tiles at the diagonal pay for the mask)
            const int lim = kv - (q0u + hl * 4);
#pragma unroll
            for (int r = 0; r < 16; ++r) s_[r] = (r >> 2) * 8 + (r & 3) < lim ? 0.f : s_[r];
        }
        f32x16 dsacc;
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const f32x4 dv4 = *(lds_f4)(stats + (TQ + rb * 32 + r4 * 8) * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) dsacc[r4 * 4 + e] = s_[r4 * 4 + e] * (p_[r4 * 4 + e] - dv4[e]);
        }
        // dV^T += dO^T P, dK^T += Q^T dS
#pragma unroll
        for (int cch = 0; cch < 2; ++cch) {
            t.accumulate(dvacc, dor, cch * 16, pack_frag(s_, cch));
            t.accumulate(dkacc, qr, cch * 16, pack_frag(dsacc, cch));
            if constexpr (TIGHT) __builtin_amdgcn_sched_barrier(0);
        }
    }
}
// The softmax statistics of a tile's queries, fetched by its first waves (one lane a query): a plain load with nothing computed
// from it until it is put into LDS (arithmetic on the value would make these waves wait for it, and for the tile loads in front of it).
template <int TQ = 64>
struct TileStats {
    static constexpr int W = TQ / 64;   // waves for each of the two
    float v;
    __device__ __forceinline__ void fetch(const AttnArgs &a, int b, int h, int q0t, int wave, int lane) {
        if (wave < 2 * W)
            v = ((wave < W ? a.lse : a.delta) + ((int64_t)b * a.Hq + h) * a.T + q0t)[(uint32_t)min(wave % W * 64 + lane, a.T - 1 - q0t)];
    }
    // queries past T: lse = +inf makes their P (and with it dS) exactly zero
    __device__ __forceinline__ void commit(float *lds, int n_valid, int wave, int lane) const {
        if (wave < W) lds[wave * 64 + lane] = wave * 64 + lane < n_valid ? v * kLog2e : INFINITY;
        else if (wave < 2 * W) lds[wave * 64 + lane] = v;
    }
};
template <int HD, int KW, int QW>
struct DkdvLds {
    static constexpr uint32_t TILE = BwdTile<HD>::rows(walk_rows(QW)), V_BYTES = BwdTile<HD>::rows(32 * KW);
    static constexpr uint32_t STATS = 8 * walk_rows(QW), STAT_OFF = 4 * TILE + V_BYTES, BYTES = STAT_OFF + 2 * STATS;
};
template <int HD, int KW, int QW, bool FAR>
__global__ __launch_bounds__(64 * KW * QW) void flash_bwd_dkdv_kernel(AttnArgs a, BlockMap map) {
    constexpr int HB = HD / 32, KB = 32 * KW, NW = KW * QW, GS = BwdTile<HD>::GS, TQ = walk_rows(QW);
    using Lds = DkdvLds<HD, KW, QW>;
    constexpr uint32_t TILE = Lds::TILE, STAGE = 2 * TILE, V_OFF = 2 * STAGE, STAT_OFF = Lds::STAT_OFF;
    extern __shared__ __attribute__((aligned(256))) bf16_t smem[];
    char *lds = reinterpret_cast<char *>(smem);

    const int T = a.T, G = a.Hq / a.Hkv, nkb = (T + KB - 1) / KB;
    int set, kvb;
    if (!decode_block(map, blockIdx.x, &set, &kvb)) return;
    if (!map.by_rank) kvb = snake8(kvb, nkb);
    const int b = set / a.Hkv, hk = set % a.Hkv;
    const int lane = threadIdx.x & 63, wave = wave_index(), l32 = lane & 31, hl = lane >> 5;
    BwdTile<HD> t;
    t.init(smem, lane);
    const int kw = wave % KW, qw = wave / KW;
    const int kv0w = kvb * KB + kw * 32, kv = kv0w + l32;

    f32x16 dvacc[HB], dkacc[HB];
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
        dvacc[hb] = zero16();
        dkacc[hb] = zero16();
    }
    const float c = scalar(a.scale * kLog2e);
    const int qt_first = (kvb * KB) / TQ, n_qt = (T + TQ - 1) / TQ - qt_first;
    const int total = G * n_qt;

    DirectTile<TQ, HD, NW, FAR, GS> tq, tdo;
    tq.init(smem, a.ldq, lane, wave);
    tdo.init(smem, a.lddo, lane, wave);
    TileStats<TQ> stats;
    int f_head = 0, f_tile = 0, n_valid = 0;
    const auto request_next = [&](uint32_t stage) {
        const int h = hk * G + f_head, q0t = (qt_first + f_tile) * TQ;
        if (++f_tile == n_qt) {
            f_tile = 0;
            ++f_head;
        }
        tq.load(stage, a.q + (int64_t)b * T * a.ldq + (int64_t)h * HD, a.ldq, q0t, T);
        tdo.load(stage + TILE, a.dout + (int64_t)b * T * a.lddo + (int64_t)h * HD, a.lddo, q0t, T);
        stats.fetch(a, b, h, q0t, wave, lane);
        n_valid = T - q0t;
    };
    const auto commit = [&](uint32_t stage) {
        stats.commit(reinterpret_cast<float *>(lds + STAT_OFF + (stage ? Lds::STATS : 0)), n_valid, wave, lane);
    };
    bf16x8 kf[HD / 16];
    {
        constexpr int VW = std::min(NW, KB / BwdTile<HD>::RPL);   // waves that fetch the values
        DirectTile<KB, HD, VW, FAR, GS> tv;
        tv.init(smem, a.ldv, lane, wave);
        if (wave < VW) tv.load(V_OFF, a.v + (int64_t)b * T * a.ldv + (int64_t)hk * HD, a.ldv, kvb * KB, T);
        request_next(0);
        const bf16_t *kp = a.k + ((int64_t)b * T + min(kv, T - 1)) * a.ldk + (int64_t)hk * HD + hl * 8;
#pragma unroll
        for (int i = 0; i < HD / 16; ++i) kf[i] = load_frag_global(kp + i * 16);
        commit(0);
    }
    tile_barrier();

    const uint32_t Vw = V_OFF + BwdTile<HD>::rows(kw * 32);
    uint32_t stat_base = lds_address(smem) + STAT_OFF + hl * 16;
    asm volatile("" : "+v"(stat_base));   // (one register, see BwdTile)
    int tq_ = 0;  // query tile inside the head
    const auto step = [&](int j, uint32_t stage) {
        const bool more = j + 1 < total;
        if (more) request_next(STAGE - stage);
        const int q0t = (qt_first + tq_) * TQ;
        if ((QW <= 2 || q0t + qw * 32 < T) && kv0w < T)
            dkdv_tile<HD, TQ / 32 / QW, HD == 128 && NW == 8, TQ>(dvacc, dkacc, kf, stage, stage + TILE, stat_base + (stage ? Lds::STATS : 0), Vw, t, qw,
                              q0t, kv0w, kv, hl, c);
        if (more) commit(STAGE - stage);
        tile_barrier();
        tq_ = tq_ + 1 == n_qt ? 0 : tq_ + 1;
    };
    for (int j = 0; j < total; j += 2) {
        step(j, 0);
        if (j + 1 < total) step(j + 1, STAGE);
    }
    if constexpr (QW == 2) {
        float *red = reinterpret_cast<float *>(smem) + kw * (HB * 16 * 64) + lane;
        auto add_halves = [&](f32x16 (&acc)[HB]) {
            if (qw == 1) {
#pragma unroll
                for (int i = 0; i < HB * 16; ++i) red[i * 64] = acc[i / 16][i % 16];
            }
            __syncthreads();
            if (qw == 0) {
#pragma unroll
                for (int i = 0; i < HB * 16; ++i) acc[i / 16][i % 16] += red[i * 64];
            }
            __syncthreads();
        };
        add_halves(dvacc);
        add_halves(dkacc);
        if (qw == 1) return;
    }
    if constexpr (QW > 2) {
        const bool valid = kv < T;
        const int64_t row = (int64_t)b * T + kv;
        const float *cs = a.rope_cos ? a.rope_cos + (int64_t)kv * (HD / 2) : nullptr, *sn = a.rope_cos ? a.rope_sin + (int64_t)kv * (HD / 2) : nullptr;
        store_summed<HD, KW, QW>(a.dk + row * a.lddk + (int64_t)hk * HD, dkacc, a.scale, kw, qw, lane, valid, cs, sn, lds);
        store_summed<HD, KW, QW>(a.dv + row * a.lddv + (int64_t)hk * HD, dvacc, 1.0f, kw, qw, lane, valid, nullptr, nullptr, lds);
        return;
    }
    if (kv0w < T) {
        const int n_valid = min(32, T - kv0w);
        write_owned_rows<HD>(a.dk + ((int64_t)b * T + kv0w) * a.lddk + (int64_t)hk * HD, a.lddk, dkacc, a.scale, l32, hl,
                             n_valid, a.rope_cos ? a.rope_cos + (int64_t)kv0w * (HD / 2) : nullptr,
                             a.rope_cos ? a.rope_sin + (int64_t)kv0w * (HD / 2) : nullptr, out_region<HD>(smem, kw));
        write_owned_rows<HD>(a.dv + ((int64_t)b * T + kv0w) * a.lddv + (int64_t)hk * HD, a.lddv, dvacc, 1.0f, l32, hl,
                             n_valid, nullptr, nullptr, out_region<HD>(smem, kw));
    }
}

// The same in blocks of 256 keys with one workgroup per compute unit that goes through a list of them (see flash_fwd_chain_kernel).  A
// wave's keys and values are its own: those of the next block are requested as soon as it is done with the present one, and come in
// while it stores its results.
// LDS: two stages of Q, dO | V | statistics | the waves' results on their way out
template <int HD>
__global__ __launch_bounds__(512) void flash_bwd_dkdv_chain_kernel(AttnArgs a, ChainMap map) {
    constexpr int HB = HD / 32, KB = 256, GS = BwdTile<HD>::GS;
    constexpr uint32_t TILE = BwdTile<HD>::BYTES, STAGE = 2 * TILE, V_OFF = 2 * STAGE, STAT_OFF = V_OFF + KB / 64 * TILE, O_OFF = STAT_OFF + 1024;
    extern __shared__ __attribute__((aligned(256))) bf16_t smem[];
    char *lds = reinterpret_cast<char *>(smem);
    const int T = a.T, G = (int)(a.Hq / a.Hkv), nt = (T + 63) / 64;
    const int lane = threadIdx.x & 63, wave = wave_index(), l32 = lane & 31, hl = lane >> 5;
    BwdTile<HD> t;
    t.init(smem, lane);
    const float c = scalar(a.scale * kLog2e);
    DirectTile<64, HD, 8, false, GS> tq, tdo;
    DirectTile<32, HD, 1, false, GS> tv;
    tq.init(smem, a.ldq, lane, wave);
    tdo.init(smem, a.lddo, lane, wave);
    tv.init(smem, a.ldv, lane, 0);
    const uint32_t Vw = V_OFF + BwdTile<HD>::rows(32) * wave;
    uint32_t stat_base = lds_address(smem) + STAT_OFF + hl * 16;
    asm volatile("" : "+v"(stat_base));   // (one register, see BwdTile)

    bf16x8 kf[HD / 16];
    TileStats<> stats;
    int n_valid = 0;
    const auto block_of = [&](const Block &blk) { return map.n_blocks - 1 - blk.qb; };   // the heaviest block is the first
    const auto request_keys = [&](const Block &blk) {
        const int k0 = block_of(blk) * KB + wave * 32;
        tv.load(Vw, a.v + (int64_t)blk.b * T * a.ldv + (int64_t)blk.h * HD, a.ldv, k0, T);
        const bf16_t *kp = a.k + ((int64_t)blk.b * T + min(k0 + l32, T - 1)) * a.ldk + (int64_t)blk.h * HD + hl * 8;
#pragma unroll
        for (int i = 0; i < HD / 16; ++i) kf[i] = load_frag_global(kp + i * 16);
    };
    const auto request_tile = [&](const Block &blk, int head, int tile, uint32_t stage) {
        const int h = blk.h * G + head, q0t = tile * 64;
        tq.load(stage, a.q + (int64_t)blk.b * T * a.ldq + (int64_t)h * HD, a.ldq, q0t, T);
        tdo.load(stage + TILE, a.dout + (int64_t)blk.b * T * a.lddo + (int64_t)h * HD, a.lddo, q0t, T);
        stats.fetch(a, blk.b, h, q0t, wave, lane);
        n_valid = T - q0t;
    };
    const auto commit = [&](uint32_t stage) { stats.commit(reinterpret_cast<float *>(lds + STAT_OFF + (stage ? 512 : 0)), n_valid, wave, lane); };

    BlockList list;
    Block cur, nxt;
    if (!list.next(map, &cur)) return;
    request_keys(cur);
    request_tile(cur, 0, block_of(cur) * (KB / 64), 0);
    commit(0);
    wave_barrier(kf);
    tile_barrier();
    while (true) {
        const bool more = list.next(map, &nxt);
        const int kvb = block_of(cur), kv0w = kvb * KB + wave * 32, kv = kv0w + l32;
        const int qt_first = kvb * (KB / 64), total = G * (nt - qt_first);
        f32x16 dvacc[HB], dkacc[HB];
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
            dvacc[hb] = zero16();
            dkacc[hb] = zero16();
        }
        int head = 0, tile = qt_first;   // of the tile at work
        const auto step = [&](int j, uint32_t stage) {
            const int tile_ = tile;
            if (++tile == nt) {
                tile = qt_first;
                ++head;
            }
            const bool here = j + 1 < total, there = !here && more && (j & 1);
            if (here) request_tile(cur, head, tile, STAGE - stage);
            if (there) request_tile(nxt, 0, block_of(nxt) * (KB / 64), STAGE - stage);
            if (j < total && kv0w < T) dkdv_tile<HD, 2, HD == 128>(dvacc, dkacc, kf, stage, stage + TILE, stat_base + (stage ? 512 : 0), Vw, t, 0, tile_ * 64, kv0w, kv, hl, c);
            if (here || there) commit(STAGE - stage);
            tile_barrier();
        };
        for (int j = 0; j < total; j += 2) {   // by twos, so that every block starts in stage 0
            step(j, 0);
            step(j + 1, STAGE);
        }
        if (more) request_keys(nxt);
        if (kv0w < T) {
            const int rows = min(32, T - kv0w), pos = min(kv, T - 1);
            const bool rope = a.rope_cos != nullptr;
            char *region = lds + O_OFF + wave * 2048;
            if (rope) rotate_back<HD>(dkacc, a.scale, hl, a.rope_cos + (int64_t)pos * (HD / 2), a.rope_sin + (int64_t)pos * (HD / 2));
            write_rows_by_parts<HD, 32>(a.dk + ((int64_t)cur.b * T + kv0w) * a.lddk + (int64_t)cur.h * HD, a.lddk, dkacc, rope ? 1.0f : a.scale, l32, hl, rows, region);
            write_rows_by_parts<HD, 32>(a.dv + ((int64_t)cur.b * T + kv0w) * a.lddv + (int64_t)cur.h * HD, a.lddv, dvacc, 1.0f, l32, hl, rows, region);
        }
        wave_barrier(kf);   // no other wave waits for these keys and values
        if (!more) break;
        cur = nxt;
    }
}

// Small problems: dQ and dK/dV side by side in one launch, each working out the row sums of dO * O for itself, so that neither waits for the other.
// What bounds them is latency: each alone leaves most of the chip idle for the 8-60 us of its longest walk.  The blocks of keys come first, theirs
// is the longer walk.
//
// A block's KW x QW waves own 32 keys each and walk pieces of 32 queries; those of all the group's heads are dealt to the QW sets in turn.  A wave
// fetches its pieces into LDS of its own, one ahead, and waits for nobody until the sets' sums are added.  A tile shared by the waves
// (flash_bwd_dkdv_kernel) holds rows of one head only and ends with a barrier: 3 x 520, 8 heads of 64 on 2, are 12 steps of it and 9 here.  The row sums
// come from the chunks of dO and O that a lane itself fetched (a fragment's layout would take 32 lines per load: 26 us against 21 of this kernel alone), added
// in dQ's order, so that both have the same delta.  OWN = false: delta is dQ's, which came before (dK, dV in the place of K, V).
// us, backward, two launches -> one: 3 x 520, 8 heads on 2, head_dim 64 30.1 -> 20.6; 7 x 128, 10 on 2 19.4 -> 15.5; 4 x 512, 2 on 2 16.5 -> 10.0;
// head_dim 128: 2 x 88, 20 on 4 22.6 -> 16.0; 1 x 560, 8 on 2 49.5 -> 47.7; 3 x 1120, 2 on 2 38.4 -> 30.3.  In the place of the inputs, both in two launches, tiles -> pieces:
// 1.04 times faster over 125 shapes, 0.94 (T of about 100, head_dim 64, 17.0 -> 18.0) to 1.3.
// LDS: a wave's two stages of Q, dO | the waves' lse * log2e, delta of 32 queries, twice | head_dim 128: V (64: the lane's values fit into registers)
template <int HD, int NW>
struct UnitLds {
    static constexpr uint32_t TILE = BwdTile<HD>::rows(32), WAVE = 4 * TILE, STAT_OFF = NW * WAVE, V_OFF = STAT_OFF + NW * 512, BYTES = V_OFF + (HD == 128 ? TILE : 0);
};
// The sum of a row's chunks, one to each of the HD / 8 lanes that fetched it, in the order of row_delta, whose lane half h has the chunks 2 ks + h: the even and
// the odd ks apart, then these two, then the halves.  The lanes are those of the chunks up to an xor, so a step is one between lanes.  head_dim 64: in all
// lanes; 128, where four chunks follow each other: in those whose chunk is one of the first four.
template <int HD>
__device__ __forceinline__ float chunk_sum(float v) {
    const auto from = [](float x, auto ctrl) { return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), decltype(ctrl)::value, 0xf, 0xf, true)); };
    uint32_t far = __builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x104, 0xf, 0x5, false);   // lane ^ 4: from + 4
    far = __builtin_amdgcn_update_dpp(far, __float_as_uint(v), 0x114, 0xf, 0xa, false);          // and from - 4
    float s = v + __uint_as_float(far);
    if constexpr (HD == 128) {
        s += from(v, std::integral_constant<int, 0x128>());                      // lane ^ 8
        s += from(__uint_as_float(far), std::integral_constant<int, 0x128>());   // lane ^ 12
    }
    s += from(s, std::integral_constant<int, 0x4e>());   // lane ^ 2
    return s + from(s, std::integral_constant<int, 0xb1>());   // lane ^ 1
}
template <int HD, int KW, int QW, bool OWN>
__device__ __forceinline__ void dkdv_units_block(const AttnArgs &a, const BlockMap &map, uint32_t id, bf16_t *smem) {
    constexpr int HB = HD / 32, GS = BwdTile<HD>::GS, LPR = HD / 8, N = 32 * LPR / 64;   // lanes of a row, chunks that a lane fetches
    using Lds = UnitLds<HD, KW * QW>;
    static_assert(HD == 64 || KW == 1, "one wave's values in LDS");
    constexpr uint32_t TILE = Lds::TILE, STAGE = 2 * TILE;
    char *lds = reinterpret_cast<char *>(smem);

    const int T = a.T, G = a.Hq / a.Hkv, nt = (T + 31) / 32, nkb = (T + 32 * KW - 1) / (32 * KW);
    int set, kvb;
    if (!decode_block(map, id, &set, &kvb)) return;
    if (!map.by_rank) kvb = snake8(kvb, nkb);
    const int b = set / a.Hkv, hk = set % a.Hkv;
    const int lane = threadIdx.x & 63, wave = wave_index(), l32 = lane & 31, hl = lane >> 5;
    BwdTile<HD> t;
    t.init(smem, lane);
    const int kw = wave % KW, qw = wave / KW, key_unit = kvb * KW + kw, kv0 = key_unit * 32, kv = kv0 + l32;
    const float c = scalar(a.scale * kLog2e);
    const uint32_t wave_lds = lds_address(smem) + wave * Lds::WAVE;
    DirectTile<32, HD, 1, false, GS> tq, tdo, to;
    tq.init(lds + wave * Lds::WAVE, a.ldq, lane, 0);
    tdo.init(lds + wave * Lds::WAVE, a.lddo, lane, 0);
    to.init(lds, a.ldo, lane, 0);

    f32x16 dvacc[HB], dkacc[HB];
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
        dvacc[hb] = zero16();
        dkacc[hb] = zero16();
    }
    bf16x8 kf[HD / 16], vf[HD / 16];
    u32x4 of[N];
    float stat = 0.f;   // lse (and, not OWN, delta in the lanes from 32 on)
    int head = key_unit < nt ? 0 : G, unit = key_unit + qw;   // of the next piece (none for keys past the end)
    const auto settle = [&]() {
        while (unit >= nt && head < G) {
            unit -= nt - key_unit;
            ++head;
        }
    };
    const auto request = [&](uint32_t stage) {
        const int h = hk * G + head, q0 = unit * 32;
        tq.load(stage, a.q + (int64_t)b * T * a.ldq + (int64_t)h * HD, a.ldq, q0, T);
        tdo.load(stage + TILE, a.dout + (int64_t)b * T * a.lddo + (int64_t)h * HD, a.lddo, q0, T);
        if constexpr (OWN) to.load_to(of, a.o + (int64_t)b * T * a.ldo + (int64_t)h * HD, a.ldo, q0, T);
        stat = (OWN || lane < 32 ? a.lse : a.delta)[((int64_t)b * a.Hq + h) * T + min(q0 + l32, T - 1)];
        __builtin_amdgcn_sched_barrier(0);
    };
    // The row sums of dO * O of a piece that has landed, from the chunks of dO and O that this lane fetched.  Of the lanes that have a row's sum one takes it for
    // load j (head_dim 128: four take two loads each).  Queries past T: lse = +inf makes their P (and with it dS) exactly zero.
    const int taker = HD == 64 ? lane & 7 : lane & 3;
    const auto commit = [&](int q0, uint32_t stage, uint32_t stats) {
        typedef __attribute__((address_space(3))) const bf16x8 *lds_frag;
        typedef __attribute__((address_space(3))) float *lds_float;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if constexpr (OWN) {
            float mine[N / 4] = {};
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const bf16x8 dof = *(lds_frag)(wave_lds + stage + TILE + j * GS + lane * 16);
                const float d = chunk_sum<HD>(dot8(dof, __builtin_bit_cast(bf16x8, of[j])));
                mine[j / 4] = taker == j % 4 ? d : mine[j / 4];
            }
            if (HD == 64 ? taker < 4 : (lane >> 2 & 3) == lane >> 4) {
#pragma unroll
                for (int m = 0; m < N / 4; ++m) *(lds_float)(stats + (32 + (m * 4 + taker) * (64 / LPR) + lane / LPR) * 4) = mine[m];
            }
        } else if (lane >= 32) {
            *(lds_float)(stats + lane * 4) = stat;
        }
        if (lane < 32) *(lds_float)(stats + lane * 4) = q0 + lane < T ? stat * kLog2e : INFINITY;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    settle();
    if (head < G) request(0);
    {
        const bf16_t *kp = a.k + ((int64_t)b * T + min(kv, T - 1)) * a.ldk + (int64_t)hk * HD + hl * 8;
        const bf16_t *vp = a.v + ((int64_t)b * T + min(kv, T - 1)) * a.ldv + (int64_t)hk * HD + hl * 8;
#pragma unroll
        for (int i = 0; i < HD / 16; ++i) {
            kf[i] = load_frag_global(kp + i * 16);
            if constexpr (HD == 64) vf[i] = load_frag_global(vp + i * 16);
        }
        if constexpr (HD == 128) {
            DirectTile<32, HD, QW, false, GS> tv;
            tv.init(smem, a.ldv, lane, wave);
            tv.load(Lds::V_OFF, a.v + (int64_t)b * T * a.ldv + (int64_t)hk * HD, a.ldv, kv0, T);
            tile_barrier();
        }
    }
    const uint32_t mine = wave * Lds::WAVE, stats = lds_address(smem) + Lds::STAT_OFF + wave * 512;
    if (head < G) commit(unit * 32, 0, stats);
    for (uint32_t stage = 0; head < G; stage ^= 1) {
        const int q0 = unit * 32;
        unit += QW;
        settle();
        const bool more = head < G;
        if (more) request(stage ? 0 : STAGE);
        dkdv_tile<HD, 1, false, 32, HD == 64>(dvacc, dkacc, kf, mine + stage * STAGE, mine + stage * STAGE + TILE, stats + stage * 256 + hl * 16, Lds::V_OFF, t, 0, q0, kv0, kv, hl, c, vf);
        if constexpr (HD == 128) {   // (in the accumulation registers: left to itself the compiler brings them back and forth, 300 moves a piece)
#pragma unroll
            for (int hb = 0; hb < HB; ++hb) asm volatile("" : "+a"(dvacc[hb]), "+a"(dkacc[hb]));
        }
        if (more) commit(unit * 32, stage ? 0 : STAGE, stats + (stage ^ 1) * 256);
    }
    const bool valid = kv < T;
    const int64_t row = (int64_t)b * T + kv;
    const float *cs = a.rope_cos ? a.rope_cos + (int64_t)kv * (HD / 2) : nullptr, *sn = a.rope_cos ? a.rope_sin + (int64_t)kv * (HD / 2) : nullptr;
    store_summed<HD, KW, QW>(a.dk + row * a.lddk + (int64_t)hk * HD, dkacc, a.scale, kw, qw, lane, valid, cs, sn, lds);
    store_summed<HD, KW, QW>(a.dv + row * a.lddv + (int64_t)hk * HD, dvacc, 1.0f, kw, qw, lane, valid, nullptr, nullptr, lds);
}
// the first n_keys workgroups take blocks of keys, the others blocks of queries
template <int HD, int DQ_QW, int DQ_KW, int KW, int QW>
__global__ __launch_bounds__(64 * KW * QW) void flash_bwd_both_kernel(AttnArgs a, BlockMap keys, BlockMap queries, int n_keys) {
    static_assert(DQ_QW * DQ_KW == KW * QW, "workgroups of one size");
    extern __shared__ __attribute__((aligned(256))) bf16_t smem[];
    if ((int)blockIdx.x < n_keys) dkdv_units_block<HD, KW, QW, true>(a, keys, blockIdx.x, smem);
    else dq_block<HD, DQ_QW, DQ_KW, false>(a, queries, blockIdx.x - n_keys, smem);
}

template <int HD, int KW, int QW>
__global__ __launch_bounds__(64 * KW * QW) void flash_bwd_pieces_kernel(AttnArgs a, BlockMap keys) {
    extern __shared__ __attribute__((aligned(256))) bf16_t smem[];
    dkdv_units_block<HD, KW, QW, false>(a, keys, blockIdx.x, smem);
}

bool attn_shape_ok(const AttnArgs &a) {
    if (a.B <= 0 || a.T <= 0 || a.Hq <= 0 || a.Hkv <= 0 || a.Hq % a.Hkv) return false;
    if (a.hd != 64 && a.hd != 128) return false;
    if (a.T & 7) return false;
    if ((int64_t)a.B * a.Hq * ((a.T + 127) / 128) > (int64_t)1 << 30) return false;
    return true;
}
bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }
// both rotary tables or none, read 16 bytes at a time
bool rope_tables_ok(const AttnArgs &a) {
    if (!a.rope_cos && !a.rope_sin) return true;
    return a.rope_cos && a.rope_sin && aligned16(a.rope_cos) && aligned16(a.rope_sin);
}

}  // namespace

template <int HD, int QW, int KW, bool FAR = false>
static hipError_t launch_fwd(const AttnArgs &a, hipStream_t s) {
    // two stages of K and V, or what the results need on their way out (out_region, the other half's sums)
    constexpr size_t lds = std::max({(size_t)2 * 2 * walk_rows(KW) * HD * sizeof(bf16_t), (size_t)QW * 32 * (HD + 8) * sizeof(bf16_t),
                                     KW == 1 ? 0 : (size_t)(KW == 2 ? 1 : KW) * QW * (HD / 32 * 16 + 2) * 64 * sizeof(float)});
    static_assert(lds <= 160 * 1024, "LDS");
    static std::atomic<bool> done{false};
    const hipError_t e = ensure_lds(&flash_fwd_kernel<HD, QW, KW, FAR>, lds, &done);
    if (e != hipSuccess) return e;
    const int G = a.Hq / a.Hkv;
    const BlockMap map = block_map(G * ((a.T + 32 * QW - 1) / (32 * QW)), a.B * a.Hkv, G);
    hipLaunchKernelGGL((flash_fwd_kernel<HD, QW, KW, FAR>), dim3(grid_blocks(map)), dim3(64 * QW * KW), lds, s, a, map);
    return hipGetLastError();
}

// the numbers that chain_block divides stay in the range of Div
static bool chain_fits(const AttnArgs &a, int per_set) {
    const BlockMap m = block_map(per_set, a.B * a.Hkv, 1);
    return (int64_t)m.n_parts * m.per_part < 65536 && a.Hkv <= 4096 && a.Hq / a.Hkv <= 4096;
}
// Blocks of rank r cost tiles(r) 64-row tiles and `start` tiles' time more.  The groups are as an even share
// allows: with p of them at work at the same time an XCD's L2 has to hold p streams of keys or queries
// (head_dim 128, forward, groups of 1 / 4 / 8 / all: 16 x 4096, 32 heads (64 parts) 988 / 995 / 988 / 852 TFLOP/s; 16 x 4096, 40 heads on 8 (16)
// 1035 / 1020 / 1010 / 977; but 7 x 1160, 33 on 11 (10) 601 / 511 / 571 / 674).
template <typename F>
static ChainMap chain_map(int per_set, int n_sets, int Hkv, int copies, int n_blocks, double start, F tiles) {
    const BlockMap m = block_map(per_set, n_sets, copies);
    const int n_slots = m.n_parts * m.per_part, n_workers = std::min(kWorkers, n_slots), p = 1 << m.log_parts;
    // Position w or cycle - 1 - w of the deal is worker w's.  One group's work by position, the first slot at position 0; the groups behind it hold the same,
    // each begins where the one before ends, and the positions at which they begin recur.  So a grouping is weighed in about per_part + 64 x 64 steps
    // (slot by slot a launch of 8192 x 72 tokens, 32 heads, took 341 us of its caller's time, now 7).  The sums are whole numbers: no rounding.
    const int cycle = 2 * n_workers;
    const auto deal = [&](int parts, double *work) {
        double change[2 * kWorkers + 1] = {}, all = 0;
        int pos = 0;
        for (int i = 0; i < m.per_part; ++i) {
            const double t = start + tiles(std::min(per_set - 1, i * p) / copies);
            const int end = pos + parts % cycle;
            all += parts / cycle * t;
            change[pos] += t;
            if (end >= cycle) change[0] += t;
            change[end >= cycle ? end - cycle : end] -= t;
            pos = end >= cycle ? end - cycle : end;
        }
        for (int i = 0; i < cycle; ++i) work[i] = (all += change[i]);
    };
    int best = 1;
    double best_t = 0;
    for (int group = 1;; group = std::min(group * 2, m.n_parts)) {
        double one[2 * kWorkers], work[2 * kWorkers], sums[2 * kWorkers] = {};
        deal(group, one);
        const int slots = group * m.per_part % cycle, n_groups = m.n_parts / group, same = std::gcd(slots, cycle), period = cycle / same;
        for (int i = 0; i < cycle; ++i) sums[i % same] += one[i];
        for (int i = 0; i < cycle; ++i) work[i] = n_groups / period * sums[i % same];
        const auto add = [&](int first) {
            for (int i = 0; i < cycle; ++i) work[(first + i) % cycle] += one[i];
        };
        for (int g = n_groups - n_groups % period; g < n_groups; ++g) add((int)((int64_t)g * slots % cycle));
        if (m.n_parts % group) {
            deal(m.n_parts % group, one);
            add((int)((int64_t)n_groups * slots % cycle));
        }
        double most = 0;
        for (int w = 0; w < n_workers; ++w) most = std::max(most, work[w] + work[cycle - 1 - w]);
        const double t = most * (1 + 0.004 * std::min(group, kWorkers));
        if (group == 1 || t < best_t) best = group, best_t = t;
        if (group == m.n_parts) break;
    }
    ChainMap c = {n_sets, per_set, m.log_parts, m.n_parts, n_slots, n_workers, {}, {}, {}, {}, {}, n_blocks};
    c.group_slots = make_div(best * m.per_part);
    c.group_size = make_div(best);
    c.last_size = make_div(m.n_parts % best ? m.n_parts % best : best);
    c.Hkv = make_div(Hkv);
    c.G = make_div(copies);
    return c;
}

// forward and dQ; dK/dV (a block's queries are walked by the head)
static ChainMap query_lists(const AttnArgs &a) {
    const int G = a.Hq / a.Hkv, nqb = (a.T + 255) / 256;
    return chain_map(G * nqb, a.B * a.Hkv, a.Hkv, G, nqb, 1.0, [&](int r) { return std::min((a.T + 63) / 64, (nqb - r) * 4); });
}
static ChainMap key_lists(const AttnArgs &a) {
    const int G = a.Hq / a.Hkv, nt = (a.T + 63) / 64, nkb = (a.T + 255) / 256;
    return chain_map(nkb, a.B * a.Hkv, a.Hkv, 1, nkb, 1.0, [&](int r) { return G * (nt - r * 4); });
}

template <int HD>
static hipError_t launch_fwd_chain(const AttnArgs &a, hipStream_t s) {
    constexpr size_t lds = 2 * 2 * 64 * HD * 2 + 256 * HD * 2 + 8 * 4096;
    static std::atomic<bool> done{false};
    const hipError_t e = ensure_lds(&flash_fwd_chain_kernel<HD>, lds, &done);
    if (e != hipSuccess) return e;
    const ChainMap c = query_lists(a);
    hipLaunchKernelGGL((flash_fwd_chain_kernel<HD>), dim3(kXcds * c.n_workers), dim3(512), lds, s, a, c);
    return hipGetLastError();
}

template <int HD, int QW, int KW, bool FAR = false>
static hipError_t launch_dq(const AttnArgs &a, hipStream_t s) {
    constexpr size_t lds = std::max({(size_t)2 * 2 * BwdTile<HD>::rows(walk_rows(KW)), (size_t)QW * 32 * (HD + 8) * sizeof(bf16_t),
                                     KW == 1 ? 0 : (size_t)(KW == 2 ? 1 : KW) * QW * (HD / 32 * 16) * 64 * sizeof(float)});
    static_assert(lds <= 160 * 1024, "LDS");
    static std::atomic<bool> done{false};
    const hipError_t e = ensure_lds(&flash_bwd_dq_kernel<HD, QW, KW, FAR>, lds, &done);
    if (e != hipSuccess) return e;
    const int G = a.Hq / a.Hkv;
    const BlockMap map = block_map(G * ((a.T + 32 * QW - 1) / (32 * QW)), a.B * a.Hkv, G);
    hipLaunchKernelGGL((flash_bwd_dq_kernel<HD, QW, KW, FAR>), dim3(grid_blocks(map)), dim3(64 * QW * KW), lds, s, a, map);
    return hipGetLastError();
}

template <int HD>
static hipError_t launch_dq_chain(const AttnArgs &a, hipStream_t s) {
    constexpr size_t lds = 2 * 2 * BwdTile<HD>::BYTES + 8 * 4096;
    static std::atomic<bool> done{false};
    const hipError_t e = ensure_lds(&flash_bwd_dq_chain_kernel<HD>, lds, &done);
    if (e != hipSuccess) return e;
    const ChainMap c = query_lists(a);
    hipLaunchKernelGGL((flash_bwd_dq_chain_kernel<HD>), dim3(kXcds * c.n_workers), dim3(512), lds, s, a, c);
    return hipGetLastError();
}

// Estimated time in us of a kernel that takes blocks of `block` queries (or keys): the walk of the heaviest block, or the work of
// all blocks on 256 compute units, or, where the blocks come by rank, the r-th block of a compute unit behind r - 1 that are at
// least as heavy (`share` < 1: two workgroups of the kernel share a compute unit).  `tile` and `full` are us per 64-row tile when
// a walk decides and when the chip is full, `start` and `start_full` per block.  Fitted to 316 shapes (T 64 .. 4096, 24 .. 768 blocks of
// 128 queries, 1 .. 8 query heads per KV head) on which the choice between the kernels comes out within 1 % of the best on average.
// `rows`: of a tile (64 or more).
struct AttnCost { int block, rows; double start, tile, start_full, full, share; };
static double attn_time(const AttnArgs &a, const AttnCost &c, bool keys) {
    const int G = a.Hq / a.Hkv, nt = (a.T + c.rows - 1) / c.rows, nb = (a.T + c.block - 1) / c.block, n_sets = a.B * a.Hkv;
    const int copies = keys ? 1 : G, per_set = copies * nb;
    const double tpb = (double)c.block / c.rows, cut = nb > 1 ? 0.5 * std::max(0.0, 1.0 - tpb) : 0.0;   // (a block's first or last tile counts whole)
    const BlockMap map = block_map(per_set, n_sets, copies);
    const auto tiles = [&](int inner) -> double {
        return keys ? (double)G * (nt - (int)((int64_t)inner * c.block / c.rows)) : (double)std::min(nt, (int)(((int64_t)(nb - inner / G) * c.block + c.rows - 1) / c.rows));
    };
    const double mean = keys ? G * (nt - (nb - 1) * tpb * 0.5 + cut) : ((nb - 1) * 0.5 * nb * tpb + nt) / nb + cut;
    double t = std::max(c.start + tiles(0) * c.tile, (double)n_sets * per_set / 256.0 * (c.start_full + mean * c.full));
    const int64_t slots = (int64_t)map.n_parts * map.per_part;
    if (slots <= kByRank)
        for (int r = 1; r * 32 < slots; ++r)
            t = std::max(t, (1 + r * c.share) * (c.start + tiles(std::min(per_set - 1, (r * 32 / map.n_parts) << map.log_parts)) * c.tile));
    return t;
}
// the first whose estimate no later one beats by 3 %
template <int N>
static int cheapest(const AttnArgs &a, const AttnCost (&costs)[N], bool keys) {
    int best = 0;
    double best_t = attn_time(a, costs[0], keys);
    for (int i = 1; i < N; ++i) {
        const double t = attn_time(a, costs[i], keys);
        if (t < 0.97 * best_t) {
            best = i;
            best_t = t;
        }
    }
    return best;
}

// Forward and dQ: blocks of 128 queries with the keys split over two sets of waves, or blocks of 256?  The former walk
// their keys in two thirds of the time but fetch K and V twice as often.  Measured, blocks of 256 -> 128, us (forward; backward with
// dK/dV as below), head_dim 128 unless said:
//   256 blocks of 128: 1 x 1024 x 32 heads 30 -> 23; 81 -> 69     1 x 2048 x 16 51 -> 37; 133 -> 108     1 x 4096 x 8 95 -> 65; 238 -> 186
//   264 .. 320: 1 x 384 x 101 15 -> 19; 52 -> 56    1 x 768 x 48 23 -> 19; 67 -> 60    1 x 1536 x 25 40 -> 30; 108 -> 93
//   512: 1 x 1024 x 64 32 -> 32; 107 -> 104    1 x 2048 x 32 55 -> 47; 159 -> 146      768: 1 x 1536 x 64 49 -> 61; 166 -> 177
// In grids beyond kByRank blocks of 256 go through lists, only that short sequences of head_dim 64 keep blocks of 128 in the forward: blocks of 128 -> lists, forward, head_dim 64: 8 x 2048 x 16 129 -> 94, 4 x 4096 x 16
// 183 -> 159, 8 x 1024 x 32 70 -> 53; head_dim 128 4 x 4096 x 32 733 -> 554.
static bool split_keys(const AttnArgs &a, bool forward) {
    static const AttnCost fwd64[] = {{256, 64, 2.89, 1.15, 2.7, 1.13, 1.0}, {128, 64, 3.18, 0.92, 1.96, 0.65, 0.55}};
    static const AttnCost dq64[] = {{256, 64, 3.4, 1.25, 3.4, 1.5, 1.0}, {128, 64, 4.0, 0.85, 4.0, 0.95, 1.0}};
    static const AttnCost hd128[] = {{256, 64, 4.0, 1.62, 4.0, 1.9, 1.0}, {128, 64, 5.2, 1.13, 5.2, 1.25, 1.0}};
    const BlockMap map = block_map(a.Hq / a.Hkv * ((a.T + 255) / 256), a.B * a.Hkv, a.Hq / a.Hkv);
    if ((int64_t)map.n_parts * map.per_part > kByRank)
        return forward && a.hd == 64 && a.T < 512 && (int64_t)a.B * a.Hq * ((a.T + 127) / 128) >= 1024;
    return cheapest(a, a.hd == 128 ? hd128 : forward ? fwd64 : dq64, false) == 1;
}

// Problems whose blocks do not fill the chip walk their rows with most of it idle.  Their blocks are cut further: 64 rows with the other side
// split over four sets of waves, or 32 rows with eight sets (head_dim 128: four, which is what LDS holds tiles for); a tile has 32 rows for every set.
// A walk takes a half to an eighth of the tiles, and what bounds it is a tile's own chain of loads, products and exponentials, 0.7-1.8 us.
// Taken where the estimate is 6 % below that of the kernel chosen by the rules above (`own`: 0, 1, 2 for blocks of 256, 128, 64).  Fitted to 400 shapes (T 64 .. 8192,
// up to 1200 blocks of 128 queries, 1 .. 8 query heads per KV head), over which the choice is within 0.6 % of the best on average, nowhere more than
// 2 % behind the former kernels, and on average faster than they by (head_dim 64, 128): forward 16 and 13 %, dQ 14 and 18 %, dK/dV 33 and 22 %.  us:
//   forward   1 x 4096, 4 heads on 1, head_dim 64 54 -> 26     1 x 2048, 4 heads, head_dim 128 43 -> 24
//   backward, with dQ, dK/dV and the row sums   3 x 520, 8 on 2, 64 57 -> 33     1 x 4096, 4 on 1, 64 316 -> 123     1 x 1024, 40 on 10, 128 124 -> 96
// One tile of 64 rows or less has nothing to share.
template <int N>
static int finer(const AttnArgs &a, const AttnCost (&costs)[N], int own, bool keys) {
    if (a.T <= 64 || (int64_t)a.B * a.Hq * ((a.T + 127) / 128) > 1200) return own;
    int best = own;
    double best_t = 0.94 * attn_time(a, costs[own], keys);
    for (int i = 3; i < N; ++i) {
        const double t = attn_time(a, costs[i], keys);
        if (t < best_t) {
            best = i;
            best_t = t;
        }
    }
    return best;
}
// What is launched: rows of a block, sets of waves that share it, and whether a workgroup per compute unit goes through a list of blocks.
// The launches below and the queries about them (flash_kernels) take it from the same three functions.
static AttnKernel kernel_of(const AttnArgs &a, int k) {
    const int sets[] = {1, 2, 2, 4, a.hd == 64 ? 8 : 4}, rows[] = {256, 128, 64, 64, 32};
    return {rows[k], sets[k], false, 0};
}

// 0: blocks of 256 queries, 1: of 128, keys split in two, 3: of 64, in four, 4: of 32, in eight (head_dim 128: four)
static int query_kernel(const AttnArgs &a, bool forward) {
    static const AttnCost fwd64[] = {{256, 64, 4.17, 1.05, 4.35, 1.41, 1.12}, {128, 64, 4.65, 0.66, 2.95, 0.73, 0.6}, {},
        {64, 128, 4.63, 0.71, 3.07, 0.73, 0.38}, {32, 256, 4.79, 0.84, 3.87, 0.96, 0.75}};
    static const AttnCost fwd128[] = {{256, 64, 5.13, 1.49, 0.0, 1.19, 1.44}, {128, 64, 6.39, 0.88, 7.49, 1.12, 1.02}, {},
        {64, 128, 6.36, 1.06, 6.59, 1.28, 0.99}, {32, 128, 5.14, 1.11, 4.84, 1.2, 0.88}};
    static const AttnCost dq64[] = {{256, 64, 5.04, 1.3, 4.93, 1.76, 1.31}, {128, 64, 5.65, 0.7, 5.84, 0.82, 1.02}, {},
        {64, 128, 5.56, 0.72, 5.1, 0.92, 0.82}, {32, 256, 5.68, 0.87, 4.81, 1.06, 0.81}};
    static const AttnCost dq128[] = {{256, 64, 7.39, 2.09, 0.0, 0.5, 1.55}, {128, 64, 8.37, 1.11, 9.85, 1.42, 1.29}, {},
        {64, 128, 8.39, 1.29, 8.5, 1.59, 1.04}, {32, 128, 5.91, 1.15, 5.79, 1.24, 0.91}};
    const int own = split_keys(a, forward) ? 1 : 0;
    return forward ? finer(a, a.hd == 64 ? fwd64 : fwd128, own, false) : finer(a, a.hd == 64 ? dq64 : dq128, own, false);
}

static AttnKernel fwd_kernel(const AttnArgs &a) {
    if (!near_pitch(a.ldk) || !near_pitch(a.ldv)) return kernel_of(a, 0);
    AttnKernel k = kernel_of(a, query_kernel(a, true));
    // (one tile of keys: nothing to fetch ahead, 5.4 us against 5.9)
    k.list = k.rows == 256 && a.T > 64 && near_pitch(a.ldq) && chain_fits(a, a.Hq / a.Hkv * ((a.T + 255) / 256));
    return k;
}

hipError_t flash_fwd(const AttnArgs &a, hipStream_t s) {
    if (!attn_shape_ok(a) || (a.ldq & 7) || (a.ldk & 7) || (a.ldv & 7) || (a.ldo & 3)) return hipErrorInvalidValue;
    if (!aligned16(a.q) || !aligned16(a.k) || !aligned16(a.v) || ((uintptr_t)a.o & 7)) return hipErrorInvalidValue;
    const AttnKernel k = fwd_kernel(a);
    switch (k.rows) {
        case 128: return a.hd == 128 ? launch_fwd<128, 4, 2>(a, s) : launch_fwd<64, 4, 2>(a, s);
        case 64: return a.hd == 128 ? launch_fwd<128, 2, 4>(a, s) : launch_fwd<64, 2, 4>(a, s);
        case 32: return a.hd == 128 ? launch_fwd<128, 1, 4>(a, s) : launch_fwd<64, 1, 8>(a, s);
        default: break;
    }
    if (k.list) return a.hd == 128 ? launch_fwd_chain<128>(a, s) : launch_fwd_chain<64>(a, s);
    if (!near_pitch(a.ldk) || !near_pitch(a.ldv)) return a.hd == 128 ? launch_fwd<128, 8, 1, true>(a, s) : launch_fwd<64, 8, 1, true>(a, s);
    return a.hd == 128 ? launch_fwd<128, 8, 1>(a, s) : launch_fwd<64, 8, 1>(a, s);
}

// lists of more than three blocks for every worker
static bool long_lists(const AttnArgs &a, int per_set) {
    const BlockMap m = block_map(per_set, a.B * a.Hkv, 1);
    return m.n_parts * m.per_part > 3 * kWorkers;
}
static AttnKernel dq_kernel(const AttnArgs &a) {
    if (!near_pitch(a.ldk) || !near_pitch(a.ldv)) return kernel_of(a, 0);
    AttnKernel k = kernel_of(a, query_kernel(a, false));
    const int per_set = a.Hq / a.Hkv * ((a.T + 255) / 256);
    // (T: as for the forward.  head_dim 64, lists of up to three blocks: 2 x 2048, 32 heads, two, 140 -> 144 us; four: 8 x 1024, 32 heads 245 -> 215)
    k.list = k.rows == 256 && a.T > 64 && chain_fits(a, per_set) && (a.hd == 128 || long_lists(a, per_set));
    return k;
}
static hipError_t flash_bwd_dq(const AttnArgs &a, hipStream_t s) {
    const AttnKernel k = dq_kernel(a);
    switch (k.rows) {
        case 128: return a.hd == 128 ? launch_dq<128, 4, 2>(a, s) : launch_dq<64, 4, 2>(a, s);
        case 64: return a.hd == 128 ? launch_dq<128, 2, 4>(a, s) : launch_dq<64, 2, 4>(a, s);
        case 32: return a.hd == 128 ? launch_dq<128, 1, 4>(a, s) : launch_dq<64, 1, 8>(a, s);
        default: break;
    }
    if (k.list) return a.hd == 128 ? launch_dq_chain<128>(a, s) : launch_dq_chain<64>(a, s);
    if (!near_pitch(a.ldk) || !near_pitch(a.ldv)) return a.hd == 128 ? launch_dq<128, 8, 1, true>(a, s) : launch_dq<64, 8, 1, true>(a, s);
    return a.hd == 128 ? launch_dq<128, 8, 1>(a, s) : launch_dq<64, 8, 1>(a, s);
}

template <int HD, int KW, int QW, bool FAR = false>
static hipError_t launch_dkdv(const AttnArgs &a, hipStream_t s) {
    constexpr int KB = 32 * KW;
    constexpr size_t lds = DkdvLds<HD, KW, QW>::BYTES;
    static_assert(lds <= 160 * 1024, "LDS");
    static_assert((size_t)KW * 32 * (HD + 8) * sizeof(bf16_t) <= lds, "room for the results on their way out");
    static_assert(QW == 1 || (size_t)(QW == 2 ? 1 : QW) * KW * (HD / 32) * 16 * 64 * sizeof(float) <= lds, "room for the other sets' sums");
    static std::atomic<bool> done{false};
    const hipError_t e = ensure_lds(&flash_bwd_dkdv_kernel<HD, KW, QW, FAR>, lds, &done);
    if (e != hipSuccess) return e;
    const BlockMap map = block_map((a.T + KB - 1) / KB, a.B * a.Hkv, 1);
    hipLaunchKernelGGL((flash_bwd_dkdv_kernel<HD, KW, QW, FAR>), dim3(grid_blocks(map)), dim3(64 * KW * QW), lds, s, a, map);
    return hipGetLastError();
}

template <int HD, int DQ_QW, int DQ_KW, int KW, int QW>
static hipError_t launch_both(const AttnArgs &a, hipStream_t s) {
    // either kind of block, and the sums of the sets that share one
    constexpr size_t lds = std::max({(size_t)UnitLds<HD, KW * QW>::BYTES, (size_t)KW * QW * (HD / 32 * 16) * 64 * sizeof(float),
                                     (size_t)2 * 2 * BwdTile<HD>::rows(walk_rows(DQ_KW)), (size_t)DQ_QW * 32 * (HD + 8) * sizeof(bf16_t)});
    static_assert(lds <= 160 * 1024, "LDS");
    static std::atomic<bool> done{false};
    const hipError_t e = ensure_lds(&flash_bwd_both_kernel<HD, DQ_QW, DQ_KW, KW, QW>, lds, &done);
    if (e != hipSuccess) return e;
    const int G = a.Hq / a.Hkv, kb = 32 * KW, qb = 32 * DQ_QW;
    const BlockMap keys = block_map((a.T + kb - 1) / kb, a.B * a.Hkv, 1), queries = block_map(G * ((a.T + qb - 1) / qb), a.B * a.Hkv, G);
    hipLaunchKernelGGL((flash_bwd_both_kernel<HD, DQ_QW, DQ_KW, KW, QW>), dim3(grid_blocks(keys) + grid_blocks(queries)), dim3(64 * KW * QW), lds, s, a, keys,
                       queries, (int)grid_blocks(keys));
    return hipGetLastError();
}
template <int HD, int KW, int QW>
static hipError_t launch_pieces(const AttnArgs &a, hipStream_t s) {
    constexpr size_t lds = std::max((size_t)UnitLds<HD, KW * QW>::BYTES, (size_t)KW * QW * (HD / 32 * 16) * 64 * sizeof(float));
    static_assert(lds <= 160 * 1024, "LDS");
    static std::atomic<bool> done{false};
    const hipError_t e = ensure_lds(&flash_bwd_pieces_kernel<HD, KW, QW>, lds, &done);
    if (e != hipSuccess) return e;
    const BlockMap keys = block_map((a.T + 32 * KW - 1) / (32 * KW), a.B * a.Hkv, 1);
    hipLaunchKernelGGL((flash_bwd_pieces_kernel<HD, KW, QW>), dim3(grid_blocks(keys)), dim3(64 * KW * QW), lds, s, a, keys);
    return hipGetLastError();
}

template <int HD>
static hipError_t launch_dkdv_chain(const AttnArgs &a, hipStream_t s) {
    constexpr size_t lds = 4 * BwdTile<HD>::BYTES + 2 * 2 * BwdTile<HD>::BYTES + 1024 + 8 * 2048;
    static std::atomic<bool> done{false};
    const hipError_t e = ensure_lds(&flash_bwd_dkdv_chain_kernel<HD>, lds, &done);
    if (e != hipSuccess) return e;
    const ChainMap c = key_lists(a);
    hipLaunchKernelGGL((flash_bwd_dkdv_chain_kernel<HD>), dim3(kXcds * c.n_workers), dim3(512), lds, s, a, c);
    return hipGetLastError();
}

// Which dK/dV kernel.  us of the backward (with dQ and the row sums) for (8, 1) / (4, 2) / (2, 2), head_dim 128:
//   1 x 1024, 40 heads on 10 KV heads 210 / 138 / 120     1 x 4096, 9 on 9 268 / 196 / 204       1 x 2048, 48 on 12 442 / 293 / 261
//   1 x 1536, 25 on 25 117 / 93 / 108                     1 x 384, 101 on 101 50 / 52 / 58       1 x 1536, 64 on 64 163 / 175 / 218
// head_dim 64, (8, 1) / (4, 2): 3 x 1000, 16 on 4 139 / 93.
// Up to 128 keys and without groups of query heads, a walk of two tiles, the halves' merge costs more than it saves: 264 heads, 128
// tokens, head_dim 128 50 / 53 / 54.
static int choose_dkdv(const AttnArgs &a) {
    static const AttnCost hd64[] = {{256, 64, 2.0, 2.05, 14.0, 2.3, 1.0}, {128, 64, 4.0, 1.22, 10.0, 1.27, 1.0}};
    static const AttnCost hd128[] = {{256, 64, 6.0, 3.32, 12.59, 3.68, 1.0}, {128, 64, 9.0, 2.05, 8.33, 1.98, 1.0}, {64, 64, 9.0, 1.57, 7.0, 1.69, 1.0}};
    if (a.T <= 128 && a.Hq == a.Hkv) return 0;
    return a.hd == 64 ? cheapest(a, hd64, true) : cheapest(a, hd128, true);
}

// 0, 1, 2: as above (blocks of 256, 128, 64 keys); 3: of 64, queries split over four sets of waves; 4: of 32, over eight (head_dim 128: four)
static int key_kernel(const AttnArgs &a) {
    static const AttnCost hd64[] = {{256, 64, 4.18, 1.75, 8.54, 1.09, 1.76}, {128, 64, 5.97, 1.03, 6.32, 1.21, 0.56}, {},
        {64, 128, 5.54, 1.15, 5.64, 1.32, 0.83}, {32, 256, 5.34, 1.35, 4.53, 1.57, 0.91}};
    static const AttnCost hd128[] = {{256, 64, 6.52, 2.72, 2.41, 0.45, 2.44}, {128, 64, 9.01, 1.56, 10.89, 2.04, 0.74}, {64, 64, 8.38, 1.24, 9.33, 1.38, 1.09},
        {64, 128, 8.78, 1.76, 8.92, 2.18, 0.86}, {32, 128, 6.25, 1.57, 6.34, 1.67, 0.95}};
    return finer(a, a.hd == 64 ? hd64 : hd128, choose_dkdv(a), true);
}

static AttnKernel dkdv_kernel(const AttnArgs &a) {
    if (!near_pitch(a.ldq) || !near_pitch(a.ldv) || !near_pitch(a.lddo)) return kernel_of(a, 0);
    AttnKernel k = kernel_of(a, key_kernel(a));
    const int nkb = (a.T + 255) / 256;
    // (lists of less than three blocks save less than they cost: 1 x 1536, 64 heads, 3 blocks 163 -> 165 us; 3.8 blocks 3 % faster,
    // 8 x 2048, 16 heads, 4 blocks 651 -> 547 together with dQ; head_dim 64, dK/dV alone 406 -> 319, but not for long sequences: 10 x 15 320,
    // 8 heads on 4 8310 -> 8480)
    k.list = k.rows == 256 && chain_fits(a, nkb) && long_lists(a, nkb) && (a.hd == 128 || a.T <= 6144);
    return k;
}
static hipError_t flash_bwd_dkdv(const AttnArgs &a, hipStream_t s) {
    const AttnKernel k = dkdv_kernel(a);
    switch (k.rows) {
        case 128: return a.hd == 128 ? launch_dkdv<128, 4, 2>(a, s) : launch_dkdv<64, 4, 2>(a, s);
        case 64:
            if (k.sets == 2) return launch_dkdv<128, 2, 2>(a, s);
            return a.hd == 128 ? launch_dkdv<128, 2, 4>(a, s) : launch_dkdv<64, 2, 4>(a, s);
        case 32: return a.hd == 128 ? launch_dkdv<128, 1, 4>(a, s) : launch_dkdv<64, 1, 8>(a, s);
        default: break;
    }
    if (k.list) return a.hd == 128 ? launch_dkdv_chain<128>(a, s) : launch_dkdv_chain<64>(a, s);
    if (!near_pitch(a.ldq) || !near_pitch(a.ldv) || !near_pitch(a.lddo))
        return a.hd == 128 ? launch_dkdv<128, 8, 1, true>(a, s) : launch_dkdv<64, 8, 1, true>(a, s);
    return a.hd == 128 ? launch_dkdv<128, 8, 1>(a, s) : launch_dkdv<64, 8, 1>(a, s);
}

// the rows of two arrays of B T rows may share memory: elements of their rows, pitches
static bool overlap(const AttnArgs &a, const bf16_t *x, int64_t ldx, int64_t cols_x, const bf16_t *y, int64_t ldy, int64_t cols_y) {
    const int64_t last = (int64_t)a.B * a.T - 1;
    const bf16_t *x0 = x + std::min<int64_t>(0, last * ldx), *x1 = x + std::max<int64_t>(0, last * ldx) + cols_x;
    const bf16_t *y0 = y + std::min<int64_t>(0, last * ldy), *y1 = y + std::max<int64_t>(0, last * ldy) + cols_y;
    return x0 < y1 && y0 < x1;
}
// dQ and dK/dV in one launch: where dK/dV takes blocks of 32 keys (head_dim 64: or of 64, shared by four sets) and dQ workgroups of the same size, up to
// kTogether workgroups.  Two launches against one, 125 shapes up to there: 1.0 to 1.8 times faster (1.27 on average);
// 700 to 1100 (with row sums that took less time): 0.88 to 1.12, slower where the walks are long (1 x 3528, 16 heads on 8 of 64, 896 workgroups 131 -> 145 us).
// Head_dim 128, where a piece's row sums take 0.6 us: only while those of the longest walk take less than dQ, which no longer comes first (5.9 us and 1.15 a tile
// of 128 rows).  us, 1 x 1120, 8 heads on 1 136 (159 in one launch), 1 x 744, 16 on 2 100 (113), 1 x 232, 16 on 2 40.4 (42.1), 3 x 616, 4 on 1 51.1 (53.2), but
// 3 x 816, 3 on 1 54.6 -> 53.5, 4 x 128, 16 on 2 27.6 -> 25.9, 1 x 2992, 4 on 2 116.0 -> 115.2.
constexpr int kTogether = 700;
constexpr double kPieceSums = 0.63;
static bool walks_pieces(const AttnArgs &a, const AttnKernel &dq, const AttnKernel &dkdv) {
    if (!(dkdv.rows == 32 || (dkdv.rows == 64 && dkdv.sets == 4 && a.hd == 64)) || dq.list || (a.hd == 128 && dq.rows != 32)) return false;
    const int64_t blocks = (int64_t)a.B * a.Hkv * ((a.T + dkdv.rows - 1) / dkdv.rows) + (int64_t)a.B * a.Hq * ((a.T + dq.rows - 1) / dq.rows);
    if (blocks > kTogether) return false;
    if (a.hd == 128 && kPieceSums * ((a.Hq / a.Hkv * ((a.T + 31) / 32) + 3) / 4) > 5.9 + 1.15 * ((a.T + 127) / 128)) return false;
    return near_pitch(a.ldk) && near_pitch(a.ldo);
}
// dK and dV may take the place of keys and values, but not while dQ reads them: dK/dV then has a launch of its own behind dQ, with the same walk, so that
// its results do not depend on where they go.
static bool apart_from_inputs(const AttnArgs &a) {
    const int64_t nq = (int64_t)a.Hq * a.hd, nkv = (int64_t)a.Hkv * a.hd;
    const auto apart = [&](const bf16_t *x, int64_t ldx) {
        return !overlap(a, x, ldx, nkv, a.k, a.ldk, nkv) && !overlap(a, x, ldx, nkv, a.v, a.ldv, nkv) && !overlap(a, x, ldx, nkv, a.q, a.ldq, nq) &&
               !overlap(a, x, ldx, nkv, a.dout, a.lddo, nq) && !overlap(a, x, ldx, nkv, a.o, a.ldo, nq);
    };
    return apart(a.dk, a.lddk) && apart(a.dv, a.lddv);
}
static hipError_t flash_bwd_both(const AttnArgs &a, const AttnKernel &dq, const AttnKernel &dkdv, hipStream_t s) {
    if (a.hd == 128) return launch_both<128, 1, 4, 1, 4>(a, s);
    switch (dq.rows) {
        case 256: return dkdv.rows == 64 ? launch_both<64, 8, 1, 2, 4>(a, s) : launch_both<64, 8, 1, 1, 8>(a, s);
        case 128: return dkdv.rows == 64 ? launch_both<64, 4, 2, 2, 4>(a, s) : launch_both<64, 4, 2, 1, 8>(a, s);
        case 64: return dkdv.rows == 64 ? launch_both<64, 2, 4, 2, 4>(a, s) : launch_both<64, 2, 4, 1, 8>(a, s);
        default: return dkdv.rows == 64 ? launch_both<64, 1, 8, 2, 4>(a, s) : launch_both<64, 1, 8, 1, 8>(a, s);
    }
}
static hipError_t flash_bwd_pieces(const AttnArgs &a, const AttnKernel &dkdv, hipStream_t s) {
    if (a.hd == 128) return launch_pieces<128, 1, 4>(a, s);
    return dkdv.rows == 64 ? launch_pieces<64, 2, 4>(a, s) : launch_pieces<64, 1, 8>(a, s);
}

hipError_t flash_bwd(const AttnArgs &a, hipStream_t s) {
    // everything that either kernel asks for, before one of them has written a result
    if (!attn_shape_ok(a) || !rope_tables_ok(a)) return hipErrorInvalidValue;
    if ((a.ldq & 7) || (a.ldk & 7) || (a.ldv & 7) || (a.ldo & 7) || (a.lddo & 7) || (a.lddq & 3) || (a.lddk & 3) || (a.lddv & 3)) return hipErrorInvalidValue;
    if (!aligned16(a.q) || !aligned16(a.k) || !aligned16(a.v) || !aligned16(a.o) || !aligned16(a.dout)) return hipErrorInvalidValue;
    if (((uintptr_t)a.dq & 7) || ((uintptr_t)a.dk & 7) || ((uintptr_t)a.dv & 7)) return hipErrorInvalidValue;
    hipError_t e;
    const int64_t nq = (int64_t)a.Hq * a.hd;
    if (overlap(a, a.dq, a.lddq, nq, a.q, a.ldq, nq) || overlap(a, a.dq, a.lddq, nq, a.dout, a.lddo, nq) || overlap(a, a.dq, a.lddq, nq, a.o, a.ldo, nq)) {
        // dq takes the place of something that dK/dV reads: it comes last
        e = attn_delta(a.delta, a.dout, a.lddo, a.o, a.ldo, a.B, a.T, a.Hq, a.hd, s);
        if (e == hipSuccess) e = flash_bwd_dkdv(a, s);
        AttnArgs with_delta = a;
        with_delta.o = nullptr;
        return e == hipSuccess ? flash_bwd_dq(with_delta, s) : e;
    }
    const AttnKernel dq = dq_kernel(a), dkdv = dkdv_kernel(a);
    const bool pieces = walks_pieces(a, dq, dkdv);
    if (pieces && apart_from_inputs(a)) return flash_bwd_both(a, dq, dkdv, s);
    e = flash_bwd_dq(a, s);
    if (e != hipSuccess) return e;
    return pieces ? flash_bwd_pieces(a, dkdv, s) : flash_bwd_dkdv(a, s);
}

void flash_kernels(const AttnArgs &a, AttnKernel (&k)[3]) {
    k[0] = fwd_kernel(a);
    k[1] = dq_kernel(a);
    k[2] = dkdv_kernel(a);
    for (int i = 0; i < 3; ++i) k[i].group = k[i].list ? (int)(i < 2 ? query_lists(a) : key_lists(a)).group_size.d : 0;
}
bool flash_bwd_together(const AttnArgs &a) { return walks_pieces(a, dq_kernel(a), dkdv_kernel(a)); }

}  // namespace mt
