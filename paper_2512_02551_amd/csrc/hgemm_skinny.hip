// Instantiates the skinny (memory-bound, small M) kernel family.
#include "hgemm_skinny.hpp"

namespace hgemm {

namespace {
#ifndef HGEMM_SKINNY_DEPTH
#define HGEMM_SKINNY_DEPTH 2
#endif
constexpr int kDepth = HGEMM_SKINNY_DEPTH;      // steps of loads a wave keeps in flight (4 KiB each)

template <int MB>
void (*any_b_kernel(bool fused))(GemmArgs)
{
    return fused ? skinny_gemm_kernel<MB, true, kDepth, 4, true> : skinny_gemm_kernel<MB, false, kDepth, 4, true>;
}

template <int WAVES>
void (*kernel_for(int mb, bool fused))(GemmArgs)
{
    switch (mb) {
        case 1: return fused ? skinny_gemm_kernel<1, true, kDepth, WAVES> : skinny_gemm_kernel<1, false, kDepth, WAVES>;
        case 2: return fused ? skinny_gemm_kernel<2, true, kDepth, WAVES> : skinny_gemm_kernel<2, false, kDepth, WAVES>;
        case 4:
            // 16 waves leave a lane 128 registers: two blocks of A at most
            if constexpr (WAVES < 16) return fused ? skinny_gemm_kernel<4, true, kDepth, WAVES> : skinny_gemm_kernel<4, false, kDepth, WAVES>;
            break;
    }
    return nullptr;
}

// Column-major B.  Chunks in flight per wave: three where the workgroup then takes at most 48 KiB of LDS (three to a compute unit: M <= 16 in
// strips of 16 rows), else two (16 x 5888 x 1920 in strips of 32 rows, 48 KiB: 7.2 us, with three chunks 7.3; 16 x 14336 x 4096 22.9, 23.6), and one
// where two do not fit the LDS.
template <int WAVES, int MB, int NR>
SkinnyTnKernel tn_kernel(bool fused)
{
    constexpr int NB = NR / 16, TWO = 2 * WAVES * 2 * (MB + NB);      // KiB of two chunks a wave
    constexpr int DEPTH = TWO <= 32 ? 3 : TWO <= 160 ? 2 : 1;
    if constexpr (skinny_tn_exists(WAVES, MB, NB, true))
        return {fused ? skinny_tn_gemm_kernel<MB, true, DEPTH, WAVES, NR> : skinny_tn_gemm_kernel<MB, false, DEPTH, WAVES, NR>, SkinnyTnLds<MB, DEPTH, WAVES, NB>::TOTAL};
    else if constexpr (skinny_tn_exists(WAVES, MB, NB, false))
        return fused ? SkinnyTnKernel{nullptr, 0} : SkinnyTnKernel{skinny_tn_gemm_kernel<MB, false, DEPTH, WAVES, NR>, SkinnyTnLds<MB, DEPTH, WAVES, NB>::TOTAL};
    else
        return {nullptr, 0};
}

template <int WAVES>
SkinnyTnKernel tn_kernel_for(int mb, bool fused, int nr)
{
    switch (mb * 100 + nr) {
        case 116: return tn_kernel<WAVES, 1, 16>(fused);
        case 132: return tn_kernel<WAVES, 1, 32>(fused);
        case 148: return tn_kernel<WAVES, 1, 48>(fused);
        case 164: return tn_kernel<WAVES, 1, 64>(fused);
        case 216: return tn_kernel<WAVES, 2, 16>(fused);
        case 232: return tn_kernel<WAVES, 2, 32>(fused);
        case 248: return tn_kernel<WAVES, 2, 48>(fused);
        case 264: return tn_kernel<WAVES, 2, 64>(fused);
        case 316: return tn_kernel<WAVES, 3, 16>(fused);
        case 332: return tn_kernel<WAVES, 3, 32>(fused);
        case 348: return tn_kernel<WAVES, 3, 48>(fused);
        case 364: return tn_kernel<WAVES, 3, 64>(fused);
        case 416: return tn_kernel<WAVES, 4, 16>(fused);
        case 432: return tn_kernel<WAVES, 4, 32>(fused);
        case 448: return tn_kernel<WAVES, 4, 48>(fused);
        case 464: return tn_kernel<WAVES, 4, 64>(fused);
    }
    return {nullptr, 0};
}
}  // namespace

// Row-major B whose rows start at any element: workgroups of 4 waves.
void (*skinny_any_b_kernel(int mb, bool fused))(GemmArgs)
{
    return mb == 1 ? any_b_kernel<1>(fused) : mb == 2 ? any_b_kernel<2>(fused) : mb == 4 ? any_b_kernel<4>(fused) : nullptr;
}

// Kernels for M <= 16 * mb (mb in {1, 2, 4}) and workgroups of 4, 8 or 16 waves, with or without the fused reduction; null for other
// values.  Row-major B:
void (*skinny_kernel(int mb, bool fused, int waves))(GemmArgs)
{
    return waves == 4 ? kernel_for<4>(mb, fused) : waves == 8 ? kernel_for<8>(mb, fused) : waves == 16 ? kernel_for<16>(mb, fused) : nullptr;
}

// Column-major B, with nr = 16, 32, 48 or 64 rows of it per workgroup.
SkinnyTnKernel skinny_tn_kernel(int mb, bool fused, int waves, int nr)
{
    return waves == 4 ? tn_kernel_for<4>(mb, fused, nr) : waves == 8 ? tn_kernel_for<8>(mb, fused, nr) : waves == 16 ? tn_kernel_for<16>(mb, fused, nr) : SkinnyTnKernel{nullptr, 0};
}

// Row-major B in strips of 32 columns, blocks of 16 * mb rows of A (mb 1 or 2), four waves.
SkinnyTnKernel skinny_tiles_kernel(int mb)
{
    if (mb == 1) return {skinny_tile_kernel<1, 2, 4, 32>, SkinnyTnLds<1, 2, 4, 2>::TOTAL};
    if (mb == 2) return {skinny_tile_kernel<2, 2, 4, 32>, SkinnyTnLds<2, 2, 4, 2>::TOTAL};
    return {nullptr, 0};
}

// Column-major B, A resident: the instance with the fewest registers whose eight waves hold all of K, for M <= 16 * mb (mb 1 or 2); null where
// none does.  Wider instances are slower on a K that a narrower one holds (32001 x 2048: 23.3 us, for 3072 24.5), two parts of
// K slower than one.
void (*skinny_strips(int mb, int64_t K))(GemmArgs)
{
    const int64_t steps = (K + 32 * kStripWaves - 1) / (32 * kStripWaves);
    if (mb == 1) {
        if (steps <= 6) return skinny_strips_kernel<1, 6, 1>;
        if (steps <= 8) return skinny_strips_kernel<1, 8, 1>;
        if (steps <= 12) return skinny_strips_kernel<1, 12, 1>;
        if (steps <= 16) return skinny_strips_kernel<1, 16, 1>;
        if (steps <= 20) return skinny_strips_kernel<1, 10, 2>;
        if (steps <= 32) return skinny_strips_kernel<1, 16, 2>;
    } else if (mb == 2) {
        if (steps <= 6) return skinny_strips_kernel<2, 6, 1>;
        if (steps <= 8) return skinny_strips_kernel<2, 8, 1>;
        if (steps <= 12) return skinny_strips_kernel<2, 12, 1>;
        if (steps <= 16) return skinny_strips_kernel<2, 8, 2>;
    }
    return nullptr;
}

}  // namespace hgemm
