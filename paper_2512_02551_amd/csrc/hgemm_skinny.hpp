// Memory-bound kernel family for skinny problems (M of a few rows, NN layout): C = A*B is then a
// stream of B through the chip (Section 4.3 of the paper observes that small problems leave the GPU
// under-used; this is the specialisation for them).
//
// What the machine wants for streaming was measured with pure-load probes: many small workgroups,
// every lane with a handful of independent 16-byte loads in flight, row segments of at least 256
// bytes, no long per-workgroup pipeline to fill and drain.  (A 32 MiB matrix is read cold in 6.3-6.7 us
// that way, against 8-12 us for 128-256 workgroups with deep private pipelines.)  So:
//
//   * grid = column strips of 128 (x) by K slabs (y); a workgroup of WAVES waves walks its slab in
//     steps of 16 * WAVES k-rows; a wave owns 16 rows of a step (wave w: rows 16 w .. 16 w + 15;
//     16-lane group g of it: rows 4 g .. 4 g + 3) and all 128 columns: four 16-byte loads per lane
//     straight into registers, DEPTH steps of them in flight;
//   * no trip through LDS and no barrier in the main loop.  v_mfma_f32_16x16x16_f16 takes 4
//     consecutive k per lane, which is what a lane has after its four loads (the same 8 columns of 4
//     consecutive rows of B) once the 4 x 8 block of halves it holds is transposed inside its own
//     registers (16 two-input byte selections); M sits on the instruction's other 16-wide side, A (a few
//     rows, cache resident) is loaded straight into registers, 8 bytes per lane and step.  Every
//     product the matrix cores form is a product A[m][k] * B[k][n] of the definition (rows of A
//     beyond M and k-rows beyond the slab are read as zeros and only ever meet each other or rows
//     that are not stored), so non-finite values stay in the elements the definition gives them;
//   * the waves' sums meet once, at the end, through LDS (four waves at a time) and are added in wave
//     order; K slabs are summed in slab order: either by the split-K reduction launch, or inside the
//     kernel by the workgroup that arrives last at a strip (FUSED), exactly as in the large-tile kernel.
//
// (An earlier form staged each 64 x 128 block of B through LDS for a transposing read and
// 16x16x32 instructions, with two barriers per step; this form is 3-30 % faster on every shape tried.)
#pragma once
#include "hgemm_mfma.hpp"

namespace hgemm {

constexpr int kSkinnyCols = 128;       // columns per workgroup

// MB = 16-row blocks of A a workgroup multiplies with every block of B it loads (M <= 16 * MB).
// ANYB: rows of B start at any element (odd N or leading dimension, any base).  Such a B used to be copied to padded rows
// first, which reads and writes all of it once more; global memory takes 16-byte loads at any element's address, so it is
// streamed where it lies (16 x 50257 x 4096: 240 -> 100 us, 1 x 50257 x 4096: 235 -> 95 us, 40 x 32001 x 2048: 64 -> 39 us;
// the rate is 4.3 TB/s against 5.6 for an aligned B: a 1 KiB run that starts off a line touches nine of them).  No load leaves the matrix: rows
// past the slab are read from its last row and replaced by zeros (what the buffer bounds check does otherwise), and the
// group of 8 columns that straddles the right edge is read from the row's last 8 elements and shifted down (N >= 8).
template <int MB, bool FUSED, int DEPTH, int WAVES, bool ANYB = false>
__global__ __launch_bounds__(64 * WAVES) void skinny_gemm_kernel(GemmArgs g)
{
    typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
    typedef unsigned int uint2v __attribute__((ext_vector_type(2)));
    constexpr int STEP = 16 * WAVES;                           // k-rows per step of the workgroup
    constexpr int PITCH = kSkinnyCols + 4;                     // floats per staged row of sums
    static_assert(WAVES % 4 == 0, "the sums meet four waves at a time");
    __shared__ __attribute__((aligned(16))) float red[4 * 16 * PITCH];

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int n0 = blockIdx.x * kSkinnyCols;
    const int split = blockIdx.y;
    const int k_lo = split * g.k_per_split;
    const int k_hi = min(g.K, k_lo + g.k_per_split);
    const int steps = (k_hi - k_lo + STEP - 1) / STEP;

    const unsigned OOB = 0x80000000u;
    const __amdgpu_buffer_rsrc_t rsrcA =
        __builtin_amdgcn_make_buffer_rsrc((void*)g.A, 0, (int)min((long long)g.M * g.lda * 2, 0x7fffffffLL), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcB =
        __builtin_amdgcn_make_buffer_rsrc((void*)g.B, 0, (int)min((long long)g.b_rows * g.ldb * 2, 0x7fffffffLL), 0x00020000);

    // lane (grp, c16): rows krow0 + STEP * step + s (s = 0..3) of B, columns n0 + 8 c16 .. + 7;
    // A[16 mb + c16][krow0 + STEP * step .. + 3]
    const int c16 = lane & 15, grp = lane >> 4;
    const int krow0 = k_lo + 16 * wave + 4 * grp;
    const bool col_ok = n0 + 8 * c16 < g.N;
    const int any_col = min(n0 + 8 * c16, g.N - 8);            // ANYB: where the lane's 16 bytes start, and the columns in front
    const int any_drop = n0 + 8 * c16 - any_col;               // of its own among them (8 and more: a lane without columns)
    const bool any_tail = n0 + kSkinnyCols > g.N;
    const int any_rows = min(k_hi, g.b_rows);
    const unsigned b_off = (unsigned)((krow0 * g.ldb + n0 + 8 * c16) * 2);
    unsigned a_off[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int m = 16 * mb + c16;
        a_off[mb] = m < g.M ? (unsigned)((m * g.lda + krow0) * 2) : OOB;
    }
    auto load_b = [&](int step, uint4v (&q)[4]) {
        if constexpr (ANYB) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int row = min(krow0 + step * STEP + s, any_rows - 1);
                __builtin_memcpy(&q[s], (const char*)g.B + (unsigned)((row * g.ldb + any_col) * 2), 16);
            }
            return;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bool ok = col_ok && krow0 + step * STEP + s < k_hi;
            q[s] = __builtin_amdgcn_raw_buffer_load_b128(rsrcB, ok ? b_off + (unsigned)((step * STEP + s) * g.ldb * 2) : OOB, 0, 0);
        }
    };
    // K is a multiple of 8 and krow0 of 4: the four k of a lane are in range together or not at all
    auto load_a = [&](int step, uint2v (&f)[MB]) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const bool ok = a_off[mb] != OOB && krow0 + step * STEP < k_hi;
            f[mb] = __builtin_amdgcn_raw_buffer_load_b64(rsrcA, ok ? a_off[mb] + (unsigned)(step * STEP * 2) : OOB, 0, 0);
        }
    };

    float4v acc[MB][8];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[mb][j] = float4v{0.f, 0.f, 0.f, 0.f};

    // set u holds step s with s % DEPTH == u (loads past the slab read zeros)
    uint4v bq[DEPTH][4];
    uint2v fa[DEPTH][MB];
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
        load_b(u, bq[u]);
        load_a(u, fa[u]);
    }
    for (int base = 0; base < steps; base += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const int step = base + u;
            if (step >= steps) break;
            if constexpr (ANYB) {
                if (any_tail) {                                // the strip at the right edge
                    typedef unsigned long long ull2 __attribute__((ext_vector_type(2)));
                    const unsigned d = 16u * (unsigned)min(any_drop, 8);
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        union { uint4v q; ull2 v; } x;
                        x.q = bq[u][s];
                        if (d >= 128u) x.v = ull2{0, 0};
                        else if (d >= 64u) x.v = ull2{x.v.y >> (d - 64u), 0};
                        else if (d > 0u) x.v = ull2{(x.v.x >> d) | (x.v.y << (64u - d)), x.v.y >> d};
                        bq[u][s] = x.q;
                    }
                }
                if (k_lo + (step + 1) * STEP > any_rows) {     // the step that reaches past the slab or past B
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        if (krow0 + step * STEP + s >= any_rows) bq[u][s] = uint4v{0, 0, 0, 0};
                }
            }
            // tb[j] = (B[k][n], B[k+1][n], B[k+2][n], B[k+3][n]) for the lane's column n = 8 c16 + j
            uint2v tb[8];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const unsigned x0 = bq[u][0][d], x1 = bq[u][1][d], x2 = bq[u][2][d], x3 = bq[u][3][d];
                tb[2 * d] = uint2v{(x0 & 0xffffu) | (x1 << 16), (x2 & 0xffffu) | (x3 << 16)};
                tb[2 * d + 1] = uint2v{(x0 >> 16) | (x1 & 0xffff0000u), (x2 >> 16) | (x3 & 0xffff0000u)};
            }
            uint2v af[MB];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) af[mb] = fa[u][mb];
            load_b(step + DEPTH, bq[u]);                     // refill this set
            load_a(step + DEPTH, fa[u]);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                union { uint2v i; half4 h; } bv;
                bv.i = tb[j];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    union { uint2v i; half4 h; } av;
                    av.i = af[mb];
                    acc[mb][j] = __builtin_amdgcn_mfma_f32_16x16x16f16(bv.h, av.h, acc[mb][j], 0, 0, 0);
                }
            }
        }
    }

    // ---- the waves' sums meet in LDS, one 16-row block of C and four waves at a time.
    // acc[mb][j][r] belongs to C[16 mb + c16][n0 + 32 grp + 8 r + j]
    const bool direct = g.splits == 1;
    float* mine = red + ((wave & 3) * 16 + c16) * PITCH + 32 * grp;
    const bool summing = t < 256;                              // summing role: one row, 8 columns
    const int orow = (t >> 4) & 15, ocol = 8 * (t & 15);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        float4v s0 = float4v{0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
        for (int w0 = 0; w0 < WAVES; w0 += 4) {
            if (mb > 0 || w0 > 0) __syncthreads();             // the previous round's sums have been read
            if (wave >= w0 && wave < w0 + 4) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    *(float4v*)(mine + 8 * r) = float4v{acc[mb][0][r], acc[mb][1][r], acc[mb][2][r], acc[mb][3][r]};
                    *(float4v*)(mine + 8 * r + 4) = float4v{acc[mb][4][r], acc[mb][5][r], acc[mb][6][r], acc[mb][7][r]};
                }
            }
            __syncthreads();
            if (summing) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float* src = red + (w * 16 + orow) * PITCH + ocol;
                    s0 += *(const float4v*)src;
                    s1 += *(const float4v*)(src + 4);
                }
            }
        }
        const int m = 16 * mb + orow, n = n0 + ocol;
        if (!summing || m >= g.M || n >= g.N) continue;
        if (direct) {
            half8 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o[e] = (_Float16)s0[e];
                o[4 + e] = (_Float16)s1[e];
            }
            store_cols(g.C + (size_t)m * g.ldc + n, o, g.N - n, g.c_wide);
        } else {
            float* dst = g.partial + ((size_t)split * g.M + m) * part_ld(g.N) + n;
            if (FUSED) {
                union { float4v f; unsigned long long u[2]; } v0, v1;
                v0.f = s0;
                v1.f = s1;
                store_agent((unsigned long long*)dst, v0.u[0]);
                store_agent((unsigned long long*)dst + 1, v0.u[1]);
                store_agent((unsigned long long*)dst + 2, v1.u[0]);
                store_agent((unsigned long long*)dst + 3, v1.u[1]);
            } else {
                *(float4v*)dst = s0;
                *(float4v*)(dst + 4) = s1;
            }
        }
    }
    if (!FUSED || direct) return;

    // Fused reduction over the K slabs of this strip: device-coherent plane stores above, then the
    // workgroup that arrives last re-reads all planes in slab order (the result does not depend on who
    // is last), rounds once and stores.  Nobody waits for anybody.
    if (!last_to_arrive(g.counters + blockIdx.x, g.splits, (int*)red, t == 0)) return;
    sum_split_planes<64 * WAVES, kSkinnyCols / 4>(g, 0, n0, g.M, t);
}

// The same family for column-major B (stored N x K, K contiguous: the layout in which frameworks keep the
// weights of a linear layer).  A workgroup owns NR = 16, 32, 48 or 64 rows of B (as many columns of C), so N / NR workgroups
// exist before K is split at all, and most problems need no split and no second launch.  Its waves take chunks of 64 k in
// turn: for each a wave copies 128 bytes of every row of B and of A into LDS of its own (8 rows a copy, chunks swizzled as in the
// large tiles), DEPTH chunks ahead, reads its fragments from there and multiplies (v_mfma_f32_16x16x32_f16), with no barrier: nobody
// else touches that LDS.  The waves' sums meet in LDS at the end and are added in wave order.  grid.y splits K further
// (planes, reduction launch or FUSED).
// Why LDS, where a 16-byte load of a row is an operand already: an operand has its 16 rows in consecutive lanes, and a load whose
// neighbouring lanes lie in different rows comes from the L2 at 38 GB/s per compute unit, one line a cycle for a quarter of it; with 8
// lanes to a row's 128 bytes it is 130 GB/s (1 MiB read by 256 workgroups, either way in registers or in LDS).  A and B together
// passed at 9.7 TB/s that way, and up to 16 rows A is as many bytes as B at NR = 16.
// What bounds it: the stream of B.  From HBM, the best kernel of any family before -> this: 1 x 4096 x 4096 9.8 (this family,
// loads that were operands) -> 7.7 us, 16 x 4096 x 4096 10.0 -> 8.4, 1 x 7296 x 7296 23.6 -> 20.8; in strips of 32 rows 16 x 5888 x 1920 9.0 -> 7.2, 16 x 14336 x
// 4096 24.8 -> 23.1; of 48 16 x 11008 x 4096 20.2 -> 19.1; from the cache 1 x 4096 x 4096 7.7 -> 4.6, 16 x 14336 x 4096 21.4 -> 18.3.  Not where K is long
// and A of 16 rows: 16 x 4096 x 11008 21.9 from HBM, split 32-row tiles 21.1 (17.9 from the cache, this 15.7).
// With more rows of A, a workgroup takes 16 MB of them (the blocks of rows of a strip follow one another, on one XCD as far as they go): what bounds it is the
// (16 MB + NR) * 2 bytes of each k that a compute unit fetches, at 57 GB/s from HBM, 110 from the cache.  From HBM / from the cache, the best
// kernel of any family before -> this: 24 x 2048 x 2048 5.7 / 5.1 -> 4.8 / 3.8 us, 64 x 2048 x 2048 7.7 / 6.7 -> 6.1 / 4.5 (by spec; packed, the shape is a row of the table), 96 x 3072 x 3072 14.6 / 11.6 -> 10.7 / 7.1,
// 48 x 8192 x 4096 18.6 / 15.0 -> 16.6 / 12.8.
// Four waves with three chunks each (48 KiB at NR = 16, three workgroups to a compute unit) are the best of 4, 8 and 16 waves and 2 to 8
// chunks: 1 x 4096 x 4096 7.8, eight waves 8.1, sixteen 8.2.  Strips are dealt so that an XCD's workgroups hold adjacent ones (see below).
// Instances for MB blocks of A and NB of B, of 16 rows each: at most 64 KiB of sums, and no more than four blocks a wave where 16 waves leave a lane 128
// registers; MB = 3 is a block of rows of A, which is never split.
constexpr bool skinny_tn_exists(int waves, int mb, int nb, bool fused)
{
    return waves * mb * nb <= 64 && (mb == 3 ? waves < 16 && !fused : waves < 16 || mb * nb <= 4);
}

template <int MB, int DEPTH, int WAVES, int NB>
struct SkinnyTnLds {                   // bytes
    static constexpr int COPIES = 2 * (MB + NB), CHUNK = COPIES * 1024, RING = DEPTH * CHUNK;      // of a wave
    static constexpr int SUMS = WAVES * MB * NB * 1024;
    static constexpr int TOTAL = WAVES * RING > SUMS ? WAVES * RING : SUMS;
    static_assert(TOTAL <= 160 * 1024 && COPIES * DEPTH <= 63, "LDS, vmcnt is 6 bits");
};

struct SkinnyTnKernel {                // an instance and its dynamic LDS
    void (*kernel)(GemmArgs);
    int lds;
};

template <int MB, bool FUSED, int DEPTH, int WAVES, int NR, bool TN>
__device__ __forceinline__ void skinny_strip(const GemmArgs& g)
{
    constexpr int NB = NR / 16;                                // 16-row blocks of B per workgroup
    typedef SkinnyTnLds<MB, DEPTH, WAVES, NB> L;
    static_assert(TN ? NR % 16 == 0 : NR == 32 && !FUSED, "rows of B");
    extern __shared__ __attribute__((aligned(1024))) char lds[];

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    // Tiles of a strip and a block of rows of A are dealt so that an XCD's workgroups hold adjacent ones, and no XCD more than an eighth of them.  (Dealt by strips, 81 of
    // them times 3 blocks are 33 for one XCD of 32 compute units: 95 x 3856 x 2840 from HBM / from the cache 15.7 / 11.6 -> 13.1 / 8.3 us, 218 x 576 x 3312 10.0 / 7.9 -> 6.9 / 5.4.)
    const int tiles = g.tiles_n * g.tiles_m, xcd = blockIdx.x & 7;
    const int tile = xcd * (tiles >> 3) + min(xcd, tiles & 7) + (blockIdx.x >> 3);
    const int strip = g.tiles_m > 1 ? tile / g.tiles_m : tile;
    const int n0 = strip * NR;
    const int m0 = g.tiles_m > 1 ? (tile - strip * g.tiles_m) * 16 * MB : 0;
    const int split = blockIdx.y;
    const int k_lo = split * g.k_per_split;
    const int k_hi = min(g.K, k_lo + g.k_per_split);
    const int steps = (k_hi - k_lo + 64 * WAVES - 1) / (64 * WAVES);

    const unsigned OOB = 0x80000000u;
    const int4v rsrcA = make_rsrc(g.A, (unsigned)min((long long)g.M * g.lda * 2, 0x7fffffffLL));
    const int4v rsrcB = make_rsrc(g.B, (unsigned)min((long long)(TN ? g.N : min(k_hi, g.b_rows)) * g.ldb * 2, 0x7fffffffLL));

    // A copy covers 8 rows of 128 bytes: lane i fills physical chunk i % 8 of row i / 8 with logical chunk p ^ (row / 2) % 8, in the second
    // copy of a block with the chunk four further.  Rows past the end and k past the slab (K is a multiple of 8) read as zeros.
    const int row8 = lane >> 3;
    const int chunk[2] = {(lane & 7) ^ (lane >> 4), (lane & 7) ^ (lane >> 4) ^ 4};
    int k = k_lo + wave * 64;                                  // of the chunk copied next
    unsigned at = 0, b_at = 0;                                 // and its distance from the first, in bytes
    unsigned a_off[MB][2], b_off[TN ? NB : 1][2];
    // Row-major B: a copy covers 16 rows of 32 columns, chunks swizzled for the transposing reads; rows past K lie past the end of B.
    const unsigned b_load = (unsigned)(16 * g.ldb * 2), b_step = (unsigned)(64 * WAVES * g.ldb * 2);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if constexpr (TN) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int n = n0 + 16 * nb + 8 * h + row8;
                b_off[nb][h] = n < g.N ? (unsigned)((n * g.ldb + k + chunk[h] * 8) * 2) : OOB;
            }
        } else {
            const int row = lane >> 2, n = n0 + 8 * ((lane & 3) ^ (((row >> 3) & 1) << 1));
            b_off[0][h] = n < g.N ? (unsigned)(((k + row) * g.ldb + n) * 2) : OOB;
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = m0 + 16 * mb + 8 * h + row8;
            a_off[mb][h] = m < g.M ? (unsigned)((m * g.lda + k + chunk[h] * 8) * 2) : OOB;
        }
    }
    const unsigned ring = __builtin_amdgcn_readfirstlane((int)lds_addr_of(lds)) + wave * L::RING;
    auto copy_chunk = [&](unsigned slot) {
        const bool ok[2] = {k + chunk[0] * 8 < k_hi, k + chunk[1] * 8 < k_hi};
        if constexpr (TN) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int h = 0; h < 2; ++h) dma16(rsrcB, ring + slot + (2 * nb + h) * 1024, ok[h] ? b_off[nb][h] + at : OOB);
        } else {
            static_for<2 * NB>([&](auto j) { dma16(rsrcB, ring + slot + decltype(j)::value * 1024, b_off[0][0] + b_at + decltype(j)::value * b_load); });
            b_at += b_step;
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int h = 0; h < 2; ++h) dma16(rsrcA, ring + slot + (2 * (NB + mb) + h) * 1024, ok[h] ? a_off[mb][h] + at : OOB);
        k += 64 * WAVES;
        at += 128 * WAVES;
    };

    // fragments: lane (grp, c16) has row c16 of a block, k = 32 ks + 8 grp .. + 7 of the chunk
    const int c16 = lane & 15, grp = lane >> 4;
    const char* const frag = lds + wave * L::RING + c16 * 128;
    const int at_ks[2] = {(grp ^ ((c16 >> 1) & 7)) * 16, ((4 + grp) ^ ((c16 >> 1) & 7)) * 16};
    // row-major B: a lane supplies four columns of rows 8 grp + c16 / 4 and + 4 of a k-step
    int tr_at[TN ? 1 : NB];
    if constexpr (!TN) {
        const int row = 8 * grp + (c16 >> 2);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int n = 16 * nb + 4 * (lane & 3), c = n >> 3;
            tr_at[nb] = wave * L::RING + row * (2 * NR) + (c ^ (((row >> 3) & 1) << 1)) * 16 + (n & 7) * 2;
        }
    }
    float4v acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = float4v{0.f, 0.f, 0.f, 0.f};

    // The last chunks are taken outside of the loop, with nothing more to copy: a copy past the end, of zeros, costs what one of B does (16 x 12288 x
    // 4096 from HBM / from the cache 21.1 / 16.2 -> 20.8 / 15.9 us, 32 x 8192 x 8192 29.5 / 21.3 -> 29.2 / 20.9).
    static_for<DEPTH>([&](auto d) { if (decltype(d)::value < steps) copy_chunk(decltype(d)::value * L::CHUNK); });
    unsigned slot = 0;
    auto take_chunk = [&](auto behind, bool more) {            // `behind` later chunks may be in flight
        wait_vmcnt<decltype(behind)::value * L::COPIES>();
        asm volatile("" ::: "memory");
        half8 fb[NB][2], fa[MB][2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                if constexpr (TN) {
                    fb[nb][ks] = *(const half8*)(frag + slot + 2 * nb * 1024 + at_ks[ks]);
                } else {
                    const char* q = lds + tr_at[nb] + slot + ks * 32 * (2 * NR);
                    union { struct { short4v lo, hi; } s; half8 h8; } v;
                    v.s.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)HGEMM_LDS(q));
                    v.s.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)HGEMM_LDS(q + 4 * (2 * NR)));
                    fb[nb][ks] = v.h8;
                }
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) fa[mb][ks] = *(const half8*)(frag + slot + 2 * (NB + mb) * 1024 + at_ks[ks]);
        }
        if (more) {
            __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));      // lgkmcnt(0): it is in registers, its place is free
            asm volatile("" ::: "memory");
            copy_chunk(slot);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[nb][ks], fa[mb][ks], acc[mb][nb], 0, 0, 0);
        slot = slot == (DEPTH - 1) * L::CHUNK ? 0 : slot + L::CHUNK;
    };
    for (int step = DEPTH; step < steps; ++step) take_chunk(ic<DEPTH - 1>{}, true);
    static_for<DEPTH>([&](auto d) {
        constexpr int left = DEPTH - 1 - decltype(d)::value;
        if (left < steps) take_chunk(ic<left>{}, false);
    });
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");

    // ---- the waves' sums meet in LDS.  acc[mb][nb][r] belongs to C[16 mb + c16][n0 + 16 nb + 4 grp + r]
    float* const red = (float*)lds;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) *(float4v*)(red + (((wave * MB + mb) * NB + nb) * 64 + lane) * 4) = acc[mb][nb];
    __syncthreads();
    const bool direct = g.splits == 1;
    // block (mb, nb) is summed by wave (mb * NB + nb) % WAVES
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            if ((mb * NB + nb) % WAVES != wave) continue;
            float4v s = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < WAVES; ++w) s += *(const float4v*)(red + (((w * MB + mb) * NB + nb) * 64 + lane) * 4);
            const int m = m0 + 16 * mb + c16, n = n0 + 16 * nb + 4 * grp;
            if (m >= g.M || n >= g.N) continue;
            if (direct) {
                half4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (_Float16)s[e];
                store_cols(g.C + (size_t)m * g.ldc + n, o, g.N - n, g.c_wide);
            } else {
                float* dst = g.partial + ((size_t)split * g.M + m) * part_ld(g.N) + n;
                if (FUSED) {
                    union { float4v f; unsigned long long u[2]; } v;
                    v.f = s;
                    store_agent((unsigned long long*)dst, v.u[0]);
                    store_agent((unsigned long long*)dst + 1, v.u[1]);
                } else {
                    *(float4v*)dst = s;
                }
            }
        }
    }
    if (!FUSED || direct) return;

    // fused reduction over the K slabs of these columns, as in skinny_gemm_kernel
    if (!last_to_arrive(g.counters + strip, g.splits, (int*)red, t == 0)) return;
    sum_split_planes<64 * WAVES, NR / 4>(g, 0, n0, g.M, t);
}

template <int MB, bool FUSED, int DEPTH, int WAVES, int NR>
__global__ __launch_bounds__(64 * WAVES) void skinny_tn_gemm_kernel(GemmArgs g)
{
    skinny_strip<MB, FUSED, DEPTH, WAVES, NR, true>(g);
}

// Row-major B: strips of 32 columns times blocks of 16 MB rows of A.  What bounds it are the same bytes, but half a cache line of each row of B, 16 rows a
// copy, comes slower than eight whole lines of a column-major one; strips of 64 columns are level with these where they fill the chip, and few problems
// have enough of them.  From HBM / from the cache, split tiles of the large family -> this: 25 x 1920 x 1920
// 6.4 / 6.1 -> 5.5 / 4.2 us, 38 x 1280 x 1280 5.9 / 5.5 -> 4.6 / 3.5, 69 x 1920 x 1920 8.2 / 7.5 -> 6.2 / 5.2, 92 x 2480 x 1664 7.2 / 6.9 -> 6.3 / 5.6.
template <int MB, int DEPTH, int WAVES, int NR>
__global__ __launch_bounds__(64 * WAVES) void skinny_tile_kernel(GemmArgs g)
{
    skinny_strip<MB, false, DEPTH, WAVES, NR, false>(g);
}

// The same for a long column-major B (an output head, a wide projection) and up to 32 rows of A: A stays in registers.  One workgroup
// of eight waves per compute unit walks strips of 16 rows of B.  The waves split K; each keeps its part of A as operands of its
// instructions (S of 32 k, P times), loads its part of a strip with 16-byte loads, asks for the next as soon as one is multiplied,
// and the eight sums of a strip meet in LDS, added in wave order by one wave (they take turns) while the others go on.
// The kernel above reads A as often as B through the L1s and has its workgroups' starts and ends in the open.
// Strips are dealt so that the 32 workgroups of an XCD (workgroup ids go round the XCDs) hold adjacent ones: a strip is 32 bytes of a
// row of C, and lines of C whose parts come from several L2s cost 5 us (16 x 50257 x 4096: 78.9 -> 73.3; a contiguous run of strips for
// each workgroup: 81).  More strips in flight than one are slower (32001 x 2048: 23.4, with two 24.7, three 26.7).
// 16 x 50257 x 4096 84 -> 72.8 us, 1 x 50257 x 4096 81 -> 68.8, 16 x 32000 x 4096 55.9 -> 47.1, 1 x 32001 x 2048 29.9 -> 23.3,
// 32 x 32001 x 2048 31.0 -> 27.7.  What bounds it up to 16 rows: the stream of B, 5.6-6.0 TB/s where a kernel that only reads gets 6.2, and
// 2 us until A is there.  With two blocks of rows B comes at 4.7 TB/s: a strip has twice the sums that meet in LDS and twice the 32-byte
// pieces of C, between the same barriers (which of the two it is was not told apart).
constexpr int kStripWaves = 8;
template <int MB, int S, int P>
__global__ __launch_bounds__(64 * kStripWaves, 2) void skinny_strips_kernel(GemmArgs g)
{
    typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
    __shared__ __attribute__((aligned(16))) float red[2][kStripWaves * MB * 256];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int kw = wave * g.k_per_split, kw_hi = min(g.K, kw + g.k_per_split);      // this wave's part of K: a multiple of 32, at most 32 * S * P
    const int strips = (g.N + 15) / 16, stride = gridDim.x;                         // the grid is a multiple of 8
    const int first = (int)((blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8);
    const unsigned OOB = 0x80000000u;
    const __amdgpu_buffer_rsrc_t rsrcA =
        __builtin_amdgcn_make_buffer_rsrc((void*)g.A, 0, (int)min((long long)g.M * g.lda * 2, 0x7fffffffLL), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcB =
        __builtin_amdgcn_make_buffer_rsrc((void*)g.B, 0, (int)min((long long)g.N * g.ldb * 2, 0x7fffffffLL), 0x00020000);
    const int c16 = lane & 15, grp = lane >> 4;
    const int k0 = kw + 8 * grp;                              // K is a multiple of 8: the eight k of a lane are in range together or not at all
    uint4v bq[S];
    union { uint4v u; half8 h; } fa[MB][P][S];
    auto load_b = [&](int strip, int part) {
        const int n = strip * 16 + c16;
        const int left = n < g.N ? kw_hi - k0 : 0;            // one comparison a load: two become branches
        const unsigned off = ((unsigned)n * (unsigned)g.ldb + (unsigned)k0) * 2u;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int k = (part * S + s) * 32;
            bq[s] = __builtin_amdgcn_raw_buffer_load_b128(rsrcB, k < left ? off + 2u * k : OOB, 0, 0);
        }
    };
    load_b(first, 0);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        const int m = 16 * mb + c16;
        const int left = m < g.M ? kw_hi - k0 : 0;
        const unsigned off = ((unsigned)m * (unsigned)g.lda + (unsigned)k0) * 2u;
#pragma unroll
        for (int s = 0; s < S * P; ++s) fa[mb][s / S][s % S].u = __builtin_amdgcn_raw_buffer_load_b128(rsrcA, 32 * s < left ? off + 64u * s : OOB, 0, 0);
    }
    for (int strip = first, turn = 0; strip < strips; strip += stride, ++turn) {
        float4v acc[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[mb] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int p = 0; p < P; ++p) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                union { uint4v i; half8 h; } b;
                b.i = bq[s];
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[mb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(b.h, fa[mb][p][s].h, acc[mb], 0, 0, 0);
            }
            load_b(p + 1 < P ? strip : strip + stride, (p + 1) % P);
        }
        // acc[mb][r] belongs to C[16 mb + c16][16 strip + 4 grp + r].  Two sets of sums: the one written here was last read before the
        // barrier of the strip in between.
        float* sums = red[turn & 1];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) *(float4v*)(sums + ((wave * MB + mb) * 64 + lane) * 4) = acc[mb];
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");      // not __syncthreads(): the next strips' loads stay in flight
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if ((turn * MB + mb) % kStripWaves != wave) continue;
            float4v sum = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < kStripWaves; ++w) sum += *(const float4v*)(sums + ((w * MB + mb) * 64 + lane) * 4);
            const int m = 16 * mb + c16, n = strip * 16 + 4 * grp;
            if (m >= g.M || n >= g.N) continue;
            half4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (_Float16)sum[e];
            store_cols(g.C + (size_t)m * g.ldc + n, o, g.N - n, g.c_wide);
        }
    }
}

}  // namespace hgemm
