// Phased MFMA kernel for large tiles (gfx950, 16 x 16 x 32 instructions, K-tiles of 64).
//
// What bounds it: the matrix cores, at the clock the chip holds under load.  The kernels of hgemm_mfma.hpp hand a
// whole K-tile from the copies to the readers at one barrier, so their copies go out in one burst per K-tile and have
// half a K-tile to land.  Here a K-tile is four units -- the upper and lower half of the A tile, the left and right half
// of the B tile -- and is multiplied in four phases, one quadrant of C (A half x B half) each.  Every phase reads one
// unit's fragments for a later phase and refills the one unit that nobody reads any more:
//
//   phase        multiplies     reads (LDS -> registers)   refills (HBM -> LDS)
//   1 of tile t  A0(t) x B0(t)  B1(t)                      A0(t+2)
//   2            A0(t) x B1(t)  A1(t)                      B0(t+2)
//   3            A1(t) x B1(t)  A0(t+1)                    B1(t+2)
//   4            A1(t) x B0(t)  B0(t+1)                    A1(t+2)
//
// so the copies flow evenly, each has six phases (one and a half K-tiles) to land in the same two buffers, every
// fragment is read once per K-tile, and every fragment is at least a phase old when it is used.  Six copies ahead also
// makes every wait a compile-time constant: a phase needs the unit that was issued six phases ago, so the copies of the
// five units since may still be in flight.
//
// Ordering.  At the barrier in front of a phase every wave has waited for its own copies of the unit that the phase
// reads (vmcnt), so the whole unit is visible behind it; and it has waited for all fragment reads but those of the
// phase just past (lgkmcnt), so the unit that was read two phases ago, which is the one refilled next, is free.
// K-tiles past the end are copied out of range, which moves zeros and keeps the counts.
//
// Measured against the best kernels of hgemm_mfma.hpp (same box, 256 x 256 tiles, N(0, 1) / sqrt(K) inputs): 4096^3
// 120.4 -> 100.6 us (1367 TFLOP/s), 8192^3 with column-major B 896 -> 789 us (1394), 16384 x 16384 x 8192 3431 -> 3186 us
// (1380), 3000 x 5120 x 5120 143 -> 122 us; 128 x 128 tiles: 1536^3 12.7 -> 12.0 us, 2048^3 20.7 -> 19.8 us.
// What is left is the chip's power limit: variants that differ in how they wait (one barrier per two phases), in who
// works (4 waves of 128 x 128 with the sums in accumulation registers), in the block order and in wave priorities
// (s_setprio around the matrix-core instructions: 1-2 % slower) all end within 1.5 % of each other on these sizes.
#pragma once
#include "hgemm_mfma.hpp"

namespace hgemm {

template <int BM_, int BN_, int WAVES_M_, int WAVES_N_>
struct PhasedCfg {      // LDS: two buffers of four units or, where that is more, the epilogue's tile: 132 KiB at 256 x 256; 64 at 128 x 128, two workgroups per compute unit
    static constexpr int BM = BM_, BN = BN_, BK = 64, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
    static constexpr int NWAVES = WAVES_M * WAVES_N, THREADS = 64 * NWAVES;
    static constexpr int HM = BM / 2, HN = BN / 2;                       // rows / columns of a unit
    static constexpr int QM = HM / WAVES_M, QN = HN / WAVES_N;           // a wave's share of a quadrant
    static constexpr int TM = QM / 16, TN = QN / 16;
    static constexpr int A_UNIT = HM * BK * 2, B_UNIT = HN * BK * 2;     // bytes
    static constexpr int A_LOADS = A_UNIT / 1024 / NWAVES, B_LOADS = B_UNIT / 1024 / NWAVES;   // copies per wave per unit
    static constexpr int B_BASE = 4 * A_UNIT;                            // LDS: A units (buffer, half), then B units
    static constexpr int B_CPR = HN / 8, B_RPI = 64 / B_CPR;             // row-major B: chunks per row, rows per wave-load
    static constexpr int OUT_PITCH = BN * 2 + 16;                        // epilogue staging: 16 rows meet 64 different banks
    static constexpr int LDS_BYTES = (4 * (A_UNIT + B_UNIT) > BM * OUT_PITCH) ? 4 * (A_UNIT + B_UNIT) : BM * OUT_PITCH;
    static_assert(QM % 16 == 0 && QN % 16 == 0, "quadrant share");
    static_assert(A_UNIT % (1024 * NWAVES) == 0 && B_UNIT % (1024 * NWAVES) == 0, "a unit splits into wave loads");
    static_assert((NWAVES * 8) % 16 == 0 && (NWAVES * B_RPI) % 16 == 0, "one swizzle serves all of a lane's copies");
    static_assert(HN == 64 || HN == 128, "row pitch of a row-major B unit");
    static_assert(4 * A_UNIT <= 65536 && 4 * B_UNIT <= 65536, "16-bit LDS offsets");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
    static_assert(3 * (A_LOADS + B_LOADS) <= 63, "vmcnt is 6 bits");
};

// SPLITK: grid.y = split, the workgroup multiplies its K range and stores fp32 sums for the split-K reduction.
template <class C, bool SPLITK, bool TN>
__global__ __launch_bounds__(C::THREADS) void phased_gemm_kernel(GemmArgs g)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    asm volatile("" :: "s"(g.A), "s"(g.B), "s"(g.C), "s"(g.M), "s"(g.N), "s"(g.K), "s"(g.lda), "s"(g.ldb), "s"(g.ldc),
                 "s"(g.tiles_m), "s"(g.tiles_n), "s"(g.swizzle), "s"(g.k_per_split), "s"(g.b_rows), "s"(g.c_wide));
    asm volatile("" :: "s"(g.by_tiles_n.m), "s"(g.by_tiles_n.l), "s"(g.by_band.m), "s"(g.by_band.l), "s"(g.by_rows.m),
                 "s"(g.by_rows.l), "s"(g.by_last_rows.m), "s"(g.by_last_rows.l));
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
    const int l16 = lane & 15, lg = lane >> 4;
    unsigned tile_m, tile_n;
    tile_coords(blockIdx.x, g, tile_m, tile_n);
    const int m0 = (int)tile_m * C::BM, n0 = (int)tile_n * C::BN;
    const int split = SPLITK ? (int)blockIdx.y : 0;
    const int k_begin = SPLITK ? split * g.k_per_split : 0;
    const int k_end = SPLITK ? min(g.K, k_begin + g.k_per_split) : g.K;
    const int KT = (k_end - k_begin + 63) / 64;

    const unsigned OOB = 0x80000000u;
    const int4v rsrcA = make_rsrc(g.A, (unsigned)min((long long)g.M * g.lda * 2, 0x7fffffffLL));
    const int4v rsrcB = make_rsrc(g.B, (unsigned)min((long long)(TN ? g.N : min(k_end, g.b_rows)) * g.ldb * 2, 0x7fffffffLL));

    // ---- copies.  Wave-load j of an A unit (TN: of a B unit) covers 8 rows of 128 bytes; lane i fills physical chunk
    // i % 8 of row i / 8 with logical chunk p ^ (row / 2) % 8.  Lanes whose chunk lies past K, and all lanes past the last
    // K-tile, get an offset that stays out of range whatever is added (row strides are below 2^31).
    const int d_row = wave * 8 + (lane >> 3);
    const int d_chunk = (lane & 7) ^ ((d_row >> 1) & 7);
    int ka = k_begin + d_chunk * 8;                                       // first k of the lane's chunk in the K-tile copied next
    unsigned va = ka < k_end ? (unsigned)(((m0 + d_row) * g.lda + ka) * 2) : OOB;
    const unsigned a_round = (unsigned)(C::NWAVES * 8 * g.lda * 2), a_half = (unsigned)(C::HM * g.lda * 2);
    // row-major B: wave-load j covers B_RPI rows of a 64 x HN unit; swizzle as in swz_b
    const int b_row = TN ? d_row : wave * C::B_RPI + lane / C::B_CPR;
    auto swz_k = [](int k) { return C::HN == 128 ? ((k & 3) << 2) ^ (((k >> 3) & 1) << 1) : (((k >> 1) & 1) << 2) ^ (((k >> 3) & 1) << 1); };
    const int b_chunk = TN ? d_chunk : (lane % C::B_CPR) ^ swz_k(b_row);
    unsigned vb0, vb1;                                          // left and right half
    if (TN) {
        vb0 = ka < k_end ? (unsigned)(((n0 + b_row) * g.ldb + ka) * 2) : OOB;
        vb1 = 0;
    } else {
        vb0 = n0 + b_chunk * 8 < g.N ? (unsigned)(((k_begin + b_row) * g.ldb + n0 + b_chunk * 8) * 2) : OOB;
        vb1 = n0 + C::HN + b_chunk * 8 < g.N ? (unsigned)(((k_begin + b_row) * g.ldb + n0 + C::HN + b_chunk * 8) * 2) : OOB;
    }
    const unsigned b_round = (unsigned)((TN ? C::NWAVES * 8 : C::NWAVES * C::B_RPI) * g.ldb * 2);
    const unsigned b_half = (unsigned)(C::HN * g.ldb * 2);      // TN only
    const unsigned b_tile = (unsigned)(64 * g.ldb * 2);         // NN only
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((int)lds_addr_of(lds)) + wave * 1024;

    auto copy_a = [&](auto buf, auto h, auto j) {
        constexpr int at = (decltype(buf)::value * 2 + decltype(h)::value) * C::A_UNIT + decltype(j)::value * C::NWAVES * 1024;
        dma16(rsrcA, lds0 + at, va + (decltype(h)::value ? a_half : 0u) + decltype(j)::value * a_round);
    };
    auto copy_b = [&](auto buf, auto h, auto j) {
        constexpr int at = C::B_BASE + (decltype(buf)::value * 2 + decltype(h)::value) * C::B_UNIT + decltype(j)::value * C::NWAVES * 1024;
        if constexpr (TN) dma16(rsrcB, lds0 + at, vb0 + (decltype(h)::value ? b_half : 0u) + decltype(j)::value * b_round);
        else dma16(rsrcB, lds0 + at, (decltype(h)::value ? vb1 : vb0) + decltype(j)::value * b_round);
    };
    auto next_k_tile = [&]() {
        ka += 64;
        va = ka < k_end ? va + 128u : OOB;
        if (TN) {
            vb0 = ka < k_end ? vb0 + 128u : OOB;
        } else {
            vb0 += b_tile;
            vb1 += b_tile;
        }
    };

    // ---- fragment reads
    half8 fa[2][C::TM][2];                                      // [half of A][block][k-step]
    half8 fb[2][C::TN][2];                                      // [register set][block][k-step]
    const int fa_row = wm * C::QM + l16, ft_row = wn * C::QN + l16;
    int pa[2], pb[TN ? 2 : C::TN];
    static_for<2>([&](auto ks) { pa[ks] = fa_row * 128 + (((4 * ks + lg) ^ ((fa_row >> 1) & 7)) * 16); });
    if constexpr (TN) {
        static_for<2>([&](auto ks) { pb[ks] = C::B_BASE + ft_row * 128 + (((4 * ks + lg) ^ ((ft_row >> 1) & 7)) * 16); });
    } else {
        const int krow = 8 * lg + (l16 >> 2);
        static_for<C::TN>([&](auto tn) {
            const int n = wn * C::QN + tn * 16 + 4 * (lane & 3);
            pb[tn] = C::B_BASE + krow * (C::HN * 2) + ((n >> 3) ^ swz_k(krow)) * 16 + (n & 7) * 2;
        });
    }
    constexpr int A_READS = 2 * C::TM, B_READS = 2 * C::TN;     // fragments (a row-major B fragment is two reads)
    auto read_a = [&](auto buf, auto h, auto r) {
        constexpr int tm = decltype(r)::value / 2, ks = decltype(r)::value % 2;
        constexpr int at = (decltype(buf)::value * 2 + decltype(h)::value) * C::A_UNIT + tm * 16 * 128;
        fa[decltype(h)::value][tm][ks] = *(const half8*)(lds + pa[ks] + at);
    };
    auto read_b = [&](auto buf, auto h, auto set, auto r) {
        constexpr int tn = decltype(r)::value / 2, ks = decltype(r)::value % 2;
        constexpr int unit = (decltype(buf)::value * 2 + decltype(h)::value) * C::B_UNIT;
        if constexpr (TN) {
            fb[decltype(set)::value][tn][ks] = *(const half8*)(lds + pb[ks] + unit + tn * 16 * 128);
        } else {
            const char* p = lds + pb[tn] + unit + ks * 32 * (C::HN * 2);
            union { struct { short4v lo, hi; } s; half8 h8; } u;
            u.s.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)HGEMM_LDS(p));
            u.s.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)HGEMM_LDS(p + 4 * (C::HN * 2)));
            fb[decltype(set)::value][tn][ks] = u.h8;
        }
    };

    float4v acc[2][2][C::TM][C::TN];                            // [half of A][half of B]
    static_for<2>([&](auto h) { static_for<2>([&](auto q) {
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j) acc[h][q][i][j] = float4v{0.f, 0.f, 0.f, 0.f};
    }); });

    // One phase: the matrix-core instructions of quadrant (ah, bh) with B's fragments in set `bset`, each followed by its
    // share of the side work: first the fragment reads, then the copies.
    constexpr int NM = 2 * C::TM * C::TN;
    constexpr int LGKM_A = A_READS > 15 ? 15 : A_READS, LGKM_B = (TN ? B_READS : 2 * B_READS) > 15 ? 15 : (TN ? B_READS : 2 * B_READS);
    auto phase = [&](auto ah, auto bh, auto bset, auto prev_reads, auto in_flight, auto nreads_tag, auto ncopies_tag, auto&& read, auto&& copy) {
        constexpr int nreads = decltype(nreads_tag)::value, ncopies = decltype(ncopies_tag)::value;
        wait_vmcnt<decltype(in_flight)::value>();
        __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (decltype(prev_reads)::value << 8) | (3 << 14));
        asm volatile("s_barrier" ::: "memory");
        static_for<NM>([&](auto ii) {
            constexpr int i = decltype(ii)::value;
            // blocks row by row, every other row backwards: consecutive instructions share an operand
            constexpr int ks = i / (C::TM * C::TN), b = i % (C::TM * C::TN), tm = b / C::TN, tn = tm & 1 ? C::TN - 1 - b % C::TN : b % C::TN;
            constexpr int H = decltype(ah)::value, Q = decltype(bh)::value, S = decltype(bset)::value;
            acc[H][Q][tm][tn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[S][tn][ks], fa[H][tm][ks], acc[H][Q][tm][tn], 0, 0, 0);
            constexpr int lo = i * (nreads + ncopies) / NM, hi = (i + 1) * (nreads + ncopies) / NM;
            static_for<hi - lo>([&](auto t) {
                constexpr int x = lo + decltype(t)::value;
                if constexpr (x < nreads) read(ic<x>{}); else copy(ic<x - nreads>{});
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // copies still allowed in flight: those of the five units issued after the one a phase reads (order A0 B0 B1 A1)
    constexpr int AL = C::A_LOADS, BL = C::B_LOADS;
    // K-tile t in buffer P: B0 in register set P, B1 in the other
    auto tile = [&](auto p_tag) {
        constexpr int P = decltype(p_tag)::value;
        typedef ic<P> X;
        typedef ic<1 - P> Y;
        phase(ic<0>{}, ic<0>{}, X{}, ic<LGKM_B>{}, ic<3 * AL + 2 * BL>{}, ic<B_READS>{}, ic<AL>{},                  // since B1(t): A1 A0' B0' B1' A1'
              [&](auto r) { read_b(ic<P>{}, ic<1>{}, Y{}, r); }, [&](auto j) { copy_a(ic<P>{}, ic<0>{}, j); });
        phase(ic<0>{}, ic<1>{}, Y{}, ic<LGKM_B>{}, ic<3 * AL + 2 * BL>{}, ic<A_READS>{}, ic<BL>{},                  // since A1(t): A0' B0' B1' A1' A0''
              [&](auto r) { read_a(ic<P>{}, ic<1>{}, r); }, [&](auto j) { copy_b(ic<P>{}, ic<0>{}, j); });
        phase(ic<1>{}, ic<1>{}, Y{}, ic<LGKM_A>{}, ic<2 * AL + 3 * BL>{}, ic<A_READS>{}, ic<BL>{},                  // since A0': B0' B1' A1' A0'' B0''
              [&](auto r) { read_a(ic<1 - P>{}, ic<0>{}, r); }, [&](auto j) { copy_b(ic<P>{}, ic<1>{}, j); });
        phase(ic<1>{}, ic<0>{}, X{}, ic<LGKM_A>{}, ic<2 * AL + 3 * BL>{}, ic<B_READS>{}, ic<AL>{},                  // since B0': B1' A1' A0'' B0'' B1''
              [&](auto r) { read_b(ic<1 - P>{}, ic<0>{}, Y{}, r); }, [&](auto j) { copy_a(ic<P>{}, ic<1>{}, j); });
        next_k_tile();
    };

    // ---- prologue: K-tiles 0 and 1 in the order of their use, then the fragments of A0(0) and B0(0)
    static_for<2>([&](auto buf) {
        static_for<AL>([&](auto j) { copy_a(buf, ic<0>{}, j); });
        static_for<BL>([&](auto j) { copy_b(buf, ic<0>{}, j); });
        static_for<BL>([&](auto j) { copy_b(buf, ic<1>{}, j); });
        static_for<AL>([&](auto j) { copy_a(buf, ic<1>{}, j); });
        next_k_tile();
    });
    wait_vmcnt<3 * (AL + BL)>();
    asm volatile("s_barrier" ::: "memory");
    static_for<A_READS>([&](auto r) { read_a(ic<0>{}, ic<0>{}, r); });
    static_for<B_READS>([&](auto r) { read_b(ic<0>{}, ic<0>{}, ic<0>{}, r); });
    __builtin_amdgcn_sched_barrier(0);

    for (int t = 0; t + 1 < KT; t += 2) {
        tile(ic<0>{});
        tile(ic<1>{});
    }
    if (KT & 1) tile(ic<0>{});

    // ---- epilogue: fp32 -> fp16 (round to nearest even), the whole tile through LDS, 16-byte stores of whole rows.
    // The copies past the end write zeros into LDS and have to be over first.
    wait_vmcnt<0>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if constexpr (SPLITK) {
        // fp32 partial sums: 16-byte stores straight from registers
        static_for<2>([&](auto h) { static_for<2>([&](auto q) {
#pragma unroll
            for (int tm = 0; tm < C::TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < C::TN; ++tn) {
                    const int m = m0 + h * C::HM + wm * C::QM + tm * 16 + l16, n = n0 + q * C::HN + wn * C::QN + tn * 16 + 4 * lg;
                    if (m < g.M && n < g.N) *(float4v*)(g.partial + ((size_t)split * g.M + m) * part_ld(g.N) + n) = acc[h][q][tm][tn];
                }
        }); });
        return;
    }
    static_for<2>([&](auto h) { static_for<2>([&](auto q) {
#pragma unroll
        for (int tm = 0; tm < C::TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < C::TN; ++tn) {
                half4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (_Float16)acc[h][q][tm][tn][e];
                *(half4*)(lds + (h * C::HM + wm * C::QM + tm * 16 + l16) * C::OUT_PITCH + (q * C::HN + wn * C::QN + tn * 16 + 4 * lg) * 2) = o;
            }
    }); });
    __syncthreads();
    constexpr int CPR = C::BN / 8;                              // 16-byte chunks per row
    auto store_chunk = [&](int j, bool wide) {
        const int idx = j * C::THREADS + (int)threadIdx.x;
        const int r = idx / CPR, ch = idx % CPR;
        const half8 v = *(const half8*)(lds + r * C::OUT_PITCH + ch * 16);
        const int m = m0 + r, n = n0 + ch * 8;
        if (m < g.M && n < g.N) store_cols(g.C + (size_t)m * g.ldc + n, v, g.N - n, wide);
    };
    if (__builtin_expect(g.c_wide != 0, 1)) {
#pragma unroll 4
        for (int j = 0; j < C::BM * CPR / C::THREADS; ++j) store_chunk(j, true);
    } else {
#pragma unroll 1
        for (int j = 0; j < C::BM * CPR / C::THREADS; ++j) store_chunk(j, false);
    }
}

}  // namespace hgemm
