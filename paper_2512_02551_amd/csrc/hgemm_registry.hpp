// Registry of compiled MFMA specialisations, filled by one function per translation unit.
#pragma once
#include <vector>

#include "hgemm_mfma.hpp"
#include "hgemm_phased.hpp"

namespace hgemm {

struct MfmaEntry {
    int bm, bn, bk, wm, wn, st, pf;
    int threads, lds_bytes;
    bool deep;                          // deep-staged configuration: only the one-tile-per-workgroup kernels exist
    void (*plain)(GemmArgs);
    void (*splitk)(GemmArgs);
    void (*plain_tn)(GemmArgs);
    void (*splitk_tn)(GemmArgs);
    void (*streamk)(GemmArgs);
    void (*streamk_tn)(GemmArgs);
    void (*splitk_fused)(GemmArgs);
    void (*splitk_fused_tn)(GemmArgs);
    void (*persist)(GemmArgs);          // null when the configuration cannot stage its epilogue in one LDS buffer
    void (*persist_tn)(GemmArgs);
    void (*acc16)(GemmArgs);            // 16-bit accumulator variant (null for the 16-wide matrix-core blocks)
    void (*acc16_tn)(GemmArgs);
    void (*fixup)(GemmArgs);
    int mi = 32;                        // side of the matrix-core output block
    // the plain kernel for a C whose rows are not whole aligned 16-byte chunks, or a row-major B of fewer rows than K
    void (*plain_any)(GemmArgs) = nullptr;
    void (*plain_any_tn)(GemmArgs) = nullptr;
    // the phased schedule of the same tile and waves (null where there is none): plain and two-launch split-K
    void (*phased)(GemmArgs) = nullptr;
    void (*phased_tn)(GemmArgs) = nullptr;
    void (*phased_splitk)(GemmArgs) = nullptr;
    void (*phased_splitk_tn)(GemmArgs) = nullptr;
    int phased_lds = 0;
    // operands at any element, read through registers (null where there is none): plain, two-launch and fused split-K
    void (*direct)(GemmArgs) = nullptr;
    void (*direct_tn)(GemmArgs) = nullptr;
    void (*direct_splitk)(GemmArgs) = nullptr;
    void (*direct_splitk_tn)(GemmArgs) = nullptr;
    void (*direct_fused)(GemmArgs) = nullptr;
    void (*direct_fused_tn)(GemmArgs) = nullptr;
    int direct_lds = 0;
    // several problems in one launch (null where there is none)
    void (*batch)(BatchArgs) = nullptr;
    void (*batch_tn)(BatchArgs) = nullptr;
    // for the cost model, filled in by registry(): 32 x 32 blocks of a wave's tile, workgroups that a compute unit holds
    int blocks_m = 0, blocks_n = 0, resident = 0;
};

template <class C> constexpr bool has_phased()
{
    return false
#define HGEMM_PHASED(bm, bn, wm, wn, st, mi) \
    || (C::BM == bm && C::BN == bn && C::BK == 64 && C::WAVES_M == wm && C::WAVES_N == wn && C::STAGES == st && C::PF == 1 && C::MI == mi)
#include "hgemm_configs.inc"
        ;
}

template <class C> constexpr bool has_batch()
{
    return false
#define HGEMM_BATCH(bm, bn, bk, wm, wn, st, pf) \
    || (C::BM == bm && C::BN == bn && C::BK == bk && C::WAVES_M == wm && C::WAVES_N == wn && C::STAGES == st && C::PF == pf && C::MI == 32)
#include "hgemm_configs.inc"
        ;
}

template <class C> constexpr bool has_direct()
{
    return false
#define HGEMM_DIRECT(bm, bn, bk, wm, wn, st, pf) \
    || (C::BM == bm && C::BN == bn && C::BK == bk && C::WAVES_M == wm && C::WAVES_N == wn && C::STAGES == st && C::PF == pf && C::MI == 32)
#include "hgemm_configs.inc"
        ;
}

template <class C, bool TN> inline void (*persist_kernel())(GemmArgs)
{
    if constexpr (C::CAN_PERSIST) return mfma_gemm_kernel<C, MODE_PERSIST, TN>;
    else return nullptr;
}

template <class C, bool TN> inline void (*acc16_kernel())(GemmArgs)
{
    if constexpr (C::MI == 32) return mfma_gemm_kernel<C, MODE_ACC16, TN>;
    else return nullptr;
}

template <class C> inline MfmaEntry make_entry()
{
    if constexpr (C::DEEP) {
        MfmaEntry e{};
        e.bm = C::BM; e.bn = C::BN; e.bk = C::BK; e.wm = C::WAVES_M; e.wn = C::WAVES_N; e.st = C::STAGES; e.pf = C::PF;
        e.threads = C::THREADS; e.lds_bytes = C::LDS_BYTES; e.deep = C::DEEP; e.mi = C::MI;
        e.plain = mfma_gemm_kernel<C, MODE_PLAIN, false>;
        e.plain_tn = mfma_gemm_kernel<C, MODE_PLAIN, true>;
        e.plain_any = mfma_gemm_kernel<C, MODE_PLAIN_ANY, false>;
        e.plain_any_tn = mfma_gemm_kernel<C, MODE_PLAIN_ANY, true>;
        return e;
    } else {
        MfmaEntry e{C::BM, C::BN, C::BK, C::WAVES_M, C::WAVES_N, C::STAGES, C::PF, C::THREADS, C::LDS_BYTES, false,
                         mfma_gemm_kernel<C, MODE_PLAIN, false>, mfma_gemm_kernel<C, MODE_SPLITK, false>,
                         mfma_gemm_kernel<C, MODE_PLAIN, true>, mfma_gemm_kernel<C, MODE_SPLITK, true>,
                         mfma_gemm_kernel<C, MODE_STREAMK, false>, mfma_gemm_kernel<C, MODE_STREAMK, true>,
                         mfma_gemm_kernel<C, MODE_SPLITK_FUSED, false>, mfma_gemm_kernel<C, MODE_SPLITK_FUSED, true>,
                         persist_kernel<C, false>(), persist_kernel<C, true>(),
                         acc16_kernel<C, false>(), acc16_kernel<C, true>(),
                         streamk_fixup_kernel<C::BM, C::BN, C::BK>};
        e.mi = C::MI;
        e.plain_any = mfma_gemm_kernel<C, MODE_PLAIN_ANY, false>;
        e.plain_any_tn = mfma_gemm_kernel<C, MODE_PLAIN_ANY, true>;
        if constexpr (has_phased<C>()) {
            typedef PhasedCfg<C::BM, C::BN, C::WAVES_M, C::WAVES_N> P;
            static_assert(P::THREADS == C::THREADS, "the phased schedule keeps the waves");
            e.phased = phased_gemm_kernel<P, false, false>;
            e.phased_tn = phased_gemm_kernel<P, false, true>;
            e.phased_splitk = phased_gemm_kernel<P, true, false>;
            e.phased_splitk_tn = phased_gemm_kernel<P, true, true>;
            e.phased_lds = P::LDS_BYTES;
        }
        if constexpr (has_direct<C>()) {
            e.direct = mfma_gemm_kernel<C, MODE_DIRECT, false>;
            e.direct_tn = mfma_gemm_kernel<C, MODE_DIRECT, true>;
            e.direct_splitk = mfma_gemm_kernel<C, MODE_DIRECT_SPLITK, false>;
            e.direct_splitk_tn = mfma_gemm_kernel<C, MODE_DIRECT_SPLITK, true>;
            e.direct_fused = mfma_gemm_kernel<C, MODE_DIRECT_FUSED, false>;
            e.direct_fused_tn = mfma_gemm_kernel<C, MODE_DIRECT_FUSED, true>;
            e.direct_lds = 2 * C::STAGE_BYTES;
        }
        if constexpr (has_batch<C>()) {
            e.batch = mfma_gemm_kernel<C, MODE_BATCH, false, BatchArgs>;
            e.batch_tn = mfma_gemm_kernel<C, MODE_BATCH, true, BatchArgs>;
        }
        return e;
    }
}

void register_chunk_0(std::vector<MfmaEntry>& out);
void register_chunk_1(std::vector<MfmaEntry>& out);
void register_chunk_2(std::vector<MfmaEntry>& out);
void register_chunk_3(std::vector<MfmaEntry>& out);
void register_chunk_4(std::vector<MfmaEntry>& out);
void register_chunk_5(std::vector<MfmaEntry>& out);
void register_chunk_6(std::vector<MfmaEntry>& out);
void register_chunk_7(std::vector<MfmaEntry>& out);

}  // namespace hgemm
