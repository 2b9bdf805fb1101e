// Host side of the C ABI declared in include/hgemm.h: plan construction (spec
// parsing, dispatch table lookup, plan-time cost model), launch, and helpers.
#include "../../include/hgemm.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "hgemm_aux.hpp"
#include "hgemm_mfma.hpp"
#include "hgemm_registry.hpp"
#include "hgemm_skinny.hpp"

namespace hgemm {

// ---------------------------------------------------------------------------
// Kernel registry: every compiled MFMA specialisation (hgemm_configs.inc), gathered from the
// translation units that instantiate them.
// ---------------------------------------------------------------------------
constexpr int64_t kLdsPerCU = 160 * 1024;
static const std::vector<MfmaEntry>& registry()
{
    static const std::vector<MfmaEntry> r = [] {
        std::vector<MfmaEntry> v;
        register_chunk_0(v); register_chunk_1(v); register_chunk_2(v); register_chunk_3(v);
        register_chunk_4(v); register_chunk_5(v); register_chunk_6(v); register_chunk_7(v);
        for (MfmaEntry& e : v) {
            const int64_t lds = (int64_t)e.st * (e.bm + e.bn) * e.bk * 2;
            const int nw = e.wm * e.wn, tm = e.bm / e.wm / 32, tn = e.bn / e.wn / 32;
            const int regs = tm * tn * 16 + (e.pf + 1) * (tm + tn) * 4 + 40;       // accumulators + fragment sets + addressing
            const int wps = std::max(1, std::min(8, 512 / std::max(regs, 64)));  // waves per SIMD the register file admits
            e.blocks_m = tm;
            e.blocks_n = tn;
            e.resident = (int)std::max<int64_t>(1, std::min<int64_t>(kLdsPerCU / lds, nw <= wps * 4 ? (wps * 4) / nw : 1));
        }
        return v;
    }();
    return r;
}

void (*skinny_kernel(int mb, bool fused, int waves))(GemmArgs);                   // hgemm_skinny.hip
SkinnyTnKernel skinny_tn_kernel(int mb, bool fused, int waves, int nr);
SkinnyTnKernel skinny_tiles_kernel(int mb);
void (*skinny_any_b_kernel(int mb, bool fused))(GemmArgs);
void (*skinny_strips(int mb, int64_t K))(GemmArgs);

constexpr int64_t kSkinnyMaxM = 64;

enum Family { FAM_GENERIC = 0, FAM_MFMA = 1, FAM_SKINNY = 2 };

struct Spec {
    Family fam = FAM_GENERIC;
    int bm = 0, bn = 0, bk = 0, wm = 0, wn = 0, st = 0;
    int pf = 1;     // register prefetch distance in k-steps
    int sk = 1;     // split-K factor
    int gm = 8;     // tile-order group height; 0 = row-major
    int tb = 0;     // 1 = transpose row-major B into the workspace first, then run the K-contiguous (TN) kernel
    int sm = 0;     // 1 = stream-K: whole waves of tiles data-parallel, the rest shared by K-tile iterations
    int fr = 0;     // 1 = split-K with the reduction fused into the kernel (last-arriving workgroup sums in split order)
    int ps = 0;     // 1 = persistent: one workgroup per compute unit walks the tiles without draining its copy pipeline
    int ac = 32;    // accumulator width: 32 = fp32 over all of K; 16 = rounded to fp16 after every 16 products
    int mi = 32;    // matrix-core output block: 32 = v_mfma_f32_32x32x16_f16, 16 = v_mfma_f32_16x16x32_f16
    int ph = 0;     // 1 = the phased schedule of this tile (hgemm_phased.hpp)
    int di = 0;     // 1 = operands read through registers, at any element's address (MODE_DIRECT)
    int wv = 4;     // skinny family: waves per workgroup (4, 8 or 16), each taking 16 k-rows of a step
    int nr = 0;     // skinny family, column-major B: rows of B (columns of C) per workgroup (16, 32, 48 or 64; 0 = as strip_rows() has it); row-major B with mr: 32
    int mr = 0;     // skinny family: rows of A per workgroup (16, 32, 48 or 64, with a row-major B 16 or 32; 0 = all of them, up to 64)
    int ra = 0;     // skinny family, column-major B: 1 = A resident in registers, one workgroup per compute unit walks strips of B
};

// K slabs of the skinny family are whole numbers of these: row-major B the 16 rows that each wave takes at a time, column-major B 32 k a wave, half of
// what it takes (all of it with A resident), so that a slab may end with half of the waves idle.  Slabs of 64 k a wave were 0.5 % faster from HBM and 1.5 % from
// the cache on 900 split problems (35 and 7 slower by more than 3 %, 81 and 136 faster); other splits than the measured rows name.
static int64_t skinny_step(const Spec& s, bool tn = false) { return (tn ? 32 : 16) * s.wv; }
// 16-row blocks of A that a kernel of the skinny family holds for up to 64 rows
static int row_blocks_of_a(int64_t M) { return M <= 16 ? 1 : M <= 32 ? 2 : 4; }
// Rows of a column-major B per workgroup where a spec does not say: one strip for every compute unit as far as that goes.  Few rows of A from HBM, all
// four widths timed on some 80 problems of each range: 16 rows up to 4096 columns (the others leave compute units idle); 4097-8192 32 rows 0.92 of
// the time of 16; 8193-12288 48 rows 0.89; 12289-16384 32 rows 0.95 (48 1.12, 64 level with 32); beyond, in several rounds, 32 rows 1.02.
// Narrower where these waves and blocks of A have no kernel of that width; strips of 16 always have one.
static int strip_rows(const Spec& s, int64_t M, int64_t N)
{
    if (s.nr || s.sk > 1) return s.nr ? s.nr : 16;
    int nr = N <= 4096 ? 16 : N <= 8192 ? 32 : N <= 12288 ? 48 : N <= 16384 ? 32 : 16;
    while (nr > 16 && !skinny_tn_exists(s.wv, s.mr ? s.mr / 16 : row_blocks_of_a(M), nr / 16, false)) nr -= 16;
    return nr;
}
static int64_t skinny_cols(const Spec& s, bool tn, int64_t M, int64_t N) { return tn ? strip_rows(s, M, N) : kSkinnyCols; }

static std::string spec_to_string(const Spec& s)
{
    char buf[160];
    if (s.fam == FAM_GENERIC) return "generic";
    if (s.fam == FAM_SKINNY) {
        snprintf(buf, sizeof buf, "skinny,sk=%d%s", s.sk, s.fr ? ",fr=1" : "");
        if (s.wv != 4) snprintf(buf + strlen(buf), sizeof buf - strlen(buf), ",wv=%d", s.wv);
        if (s.nr) snprintf(buf + strlen(buf), sizeof buf - strlen(buf), ",nr=%d", s.nr);
        if (s.mr) snprintf(buf + strlen(buf), sizeof buf - strlen(buf), ",mr=%d", s.mr);
        if (s.ra) snprintf(buf + strlen(buf), sizeof buf - strlen(buf), ",ra=1");
        return buf;
    }
    snprintf(buf, sizeof buf, "mfma,bm=%d,bn=%d,bk=%d,wm=%d,wn=%d,st=%d,pf=%d,sk=%d,gm=%d%s", s.bm, s.bn, s.bk, s.wm, s.wn,
             s.st, s.pf, s.sk, s.gm, s.tb ? ",tb=1" : "");
    if (s.sm) strncat(buf, ",sm=1", sizeof buf - strlen(buf) - 1);
    if (s.fr) strncat(buf, ",fr=1", sizeof buf - strlen(buf) - 1);
    if (s.ps) strncat(buf, ",ps=1", sizeof buf - strlen(buf) - 1);
    if (s.ac == 16) strncat(buf, ",ac=16", sizeof buf - strlen(buf) - 1);
    if (s.mi == 16) strncat(buf, ",mi=16", sizeof buf - strlen(buf) - 1);
    if (s.ph) strncat(buf, ",ph=1", sizeof buf - strlen(buf) - 1);
    if (s.di) strncat(buf, ",di=1", sizeof buf - strlen(buf) - 1);
    return buf;
}

// Reads a spec string in place: planning a call parses one (a table row), so nothing is allocated here.
static bool parse_spec(const char* text, Spec* out)
{
    if (!text) return false;
    Spec sp;
    const char* p = text;
    auto word = [&](const char* w) {
        const size_t n = strlen(w);
        if (strncmp(p, w, n) || (p[n] != '\0' && p[n] != ',')) return false;
        p += n;
        return true;
    };
    if (word("mfma")) sp.fam = FAM_MFMA;
    else if (word("skinny")) sp.fam = FAM_SKINNY;
    else if (word("generic")) sp.fam = FAM_GENERIC;
    else return false;
    int ignored = 0;
    sp.nr = -1;                                                // not given
    const struct { char key[4]; int* value; } keys[] = {
        {"bm", &sp.bm}, {"bn", &sp.bn}, {"bk", &sp.bk}, {"wm", &sp.wm}, {"wn", &sp.wn}, {"st", &sp.st}, {"pf", &sp.pf}, {"sk", &sp.sk},
        {"gm", &sp.gm}, {"tb", &sp.tb}, {"sm", &sp.sm}, {"fr", &sp.fr}, {"ps", &sp.ps}, {"ac", &sp.ac}, {"mi", &sp.mi}, {"ph", &sp.ph},
        {"di", &sp.di}, {"wv", &sp.wv}, {"nr", &sp.nr}, {"mr", &sp.mr}, {"ra", &sp.ra},
        {"pad", &ignored},      // reported by hgemm_plan_describe; padding follows from the shape, not from the spec
    };
    while (*p) {
        ++p;                                                   // the comma in front of a key
        const char* eq = p;
        while (*eq && *eq != '=' && *eq != ',') ++eq;
        const size_t len = (size_t)(eq - p);
        if (*eq != '=' || len == 0 || eq[1] == '\0' || eq[1] == ',') return false;
        char* end = nullptr;
        const long v = strtol(eq + 1, &end, 10);
        if ((*end != '\0' && *end != ',') || v < 0 || v > (1 << 20)) return false;
        bool known = false;
        for (const auto& k : keys)
            if (strlen(k.key) == len && !strncmp(k.key, p, len)) { *k.value = (int)v; known = true; break; }
        if (!known) return false;
        p = end;
    }
    if (sp.sk < 1 || sp.tb > 1 || sp.sm > 1 || sp.fr > 1 || sp.ps > 1 || (sp.sm && sp.sk > 1) || (sp.ps && (sp.sk > 1 || sp.sm)))
        return false;
    // the 16-bit accumulator is a running sum over all of K in k order: one tile per workgroup, no splitting of K
    if ((sp.ac != 32 && sp.ac != 16) || (sp.ac == 16 && (sp.fam != FAM_MFMA || sp.sk > 1 || sp.sm || sp.ps || sp.fr))) return false;
    if (sp.mi != 32 && sp.mi != 16) return false;
    if (sp.ph > 1 || (sp.ph && (sp.fam != FAM_MFMA || sp.sm || sp.fr || sp.ps || sp.tb || sp.ac == 16))) return false;
    if (sp.di > 1 || (sp.di && (sp.fam != FAM_MFMA || sp.sm || sp.ps || sp.tb || sp.ph || sp.ac == 16 || sp.mi != 32))) return false;
    if ((sp.wv != 4 && sp.wv != 8 && sp.wv != 16) || (sp.wv != 4 && sp.fam != FAM_SKINNY)) return false;
    if (sp.nr != -1 && (sp.nr < 16 || sp.nr > 64 || sp.nr % 16 || (sp.nr != 16 && sp.fam != FAM_SKINNY))) return false;
    if (sp.nr == -1 || sp.fam != FAM_SKINNY) sp.nr = 0;
    if (sp.mr && (sp.mr < 16 || sp.mr > 64 || sp.mr % 16 || sp.fam != FAM_SKINNY || sp.sk > 1 || sp.ra)) return false;      // K is not split across workgroups too
    if (sp.ra > 1 || (sp.ra && (sp.fam != FAM_SKINNY || sp.wv != kStripWaves || (sp.nr != 0 && sp.nr != 16) || sp.sk > 1))) return false;
    *out = sp;
    return true;
}

// The configuration with square tiles of this side that also takes several problems in one launch.
static const MfmaEntry* batch_entry(int tile)
{
    for (const MfmaEntry& e : registry())
        if (e.batch && e.bm == tile && e.bn == tile) return &e;
    return nullptr;
}

static const MfmaEntry* find_entry(const Spec& s)
{
    for (const MfmaEntry& e : registry())
        if (e.bm == s.bm && e.bn == s.bn && e.bk == s.bk && e.wm == s.wm && e.wn == s.wn && e.st == s.st && e.pf == s.pf && e.mi == s.mi) return &e;
    return nullptr;
}

}  // namespace hgemm

using namespace hgemm;

struct hgemm_plan_s {
    int64_t M, N, K;
    hgemm_layouts_t lay;        // with packed leading dimensions resolved
    Spec spec;
    const MfmaEntry* entry;     // null for the generic and skinny families
    void (*skinny)(GemmArgs);   // the skinny family's kernel, else null, and its dynamic LDS
    int skinny_lds;
    void (*kernel)(GemmArgs);   // the large-tile family's main kernel and its dynamic LDS
    void (*kernel_any)(GemmArgs);   // what runs in its place for a narrow C or a B of fewer rows than K (the same, or its twin)
    int kernel_lds;
    GemmArgs args;              // pointers filled in at run time
    void* workspace;            // [transposed B (when spec.tb)] [split-K / stream-K partial sums]
    size_t workspace_bytes;
    size_t partial_offset;      // byte offset of the partial sums inside the workspace
    bool tn_kernel;             // the MFMA kernel reads B with K contiguous
    int device;
    // Problems whose N, K or leading dimensions are not multiples of 8.  The kernels store C at any width and address,
    // but read A and B in aligned 16-byte chunks: an operand whose rows do not consist of those is first copied into
    // the workspace, packed and zero-filled to multiples of 8 (the zero padding of Section 5.2).  K above is then
    // rounded up to 8 (zero columns of the copy of A make the extra products vanish), lay describes the operands as the
    // kernels see them, and the fields below keep the caller's problem.  An operand that can be read where it lies is;
    // its place in the workspace is kept all the same (`spare`), for calls whose base pointer is not 16-byte aligned, unless
    // there is no memory for it: such calls then take the generic kernel.
    // Smaller problems don't take this way: kernels that load A and B through registers read them where they lie (direct_choice).
    // Measured against copying A, B and C always, two bytes per lane (us): 1000 x 1001 x 1003 26.3 -> 10.9 (A and B
    // copied, in one launch), 16 x 50257 x 4096 with column-major B 383 -> 89 (nothing copied), with row-major B 402 -> 240
    // (and 100 by the streaming family, which reads any row-major B where it lies).
    bool padded;
    bool copy_a, copy_b;
    bool spare;                 // the workspace has room for copies of operands that are not copied otherwise
    bool copy_c;                // C's rows are 2^31 elements apart or more, which the kernels cannot address: stored packed, copied from there
    bool any_b;                 // row-major B off the 16-byte grid that the streaming family reads where it lies (never copied)
    int64_t uN, uK;
    hgemm_layouts_t ulay;
    size_t a_off, b_off, c_off; // byte offsets of the padded copies of A and B and of the packed C inside the workspace
    size_t bt_off;              // byte offset of the transposed copy of B (spec.tb)
    bool static_ws;             // the workspace is this device's static scratch array, not an allocation
    bool planned;               // the library chose the specialisation (hgemm_plan, not hgemm_plan_override)
    // Operands beyond the reach of the kernels' 32-bit buffer offsets (2 GiB per operand): the problem runs
    // as a grid of row blocks of A and C by column panels of B and C, each an ordinary plan of its own on
    // offset pointers.  A row-major B of that size cannot be cut into panels that way (a panel still spans
    // all K rows), so it is first copied, transposed, into the workspace (N x K, K contiguous), whose
    // panels of rows are contiguous.
    bool blocked = false;
    bool blocked_bt = false;            // B is row-major and goes through the transposed copy
    int64_t block_m = 0, block_n = 0;   // rows and columns per block
    hgemm_layouts_t block_lay;          // layouts the blocks' plans were made for
    hgemm_plan_s* sub[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};   // [last, shorter row block][last, narrower panel]
};

// ---------------------------------------------------------------------------
// Static scratch for hgemm_run_static(): callers that may not allocate (code under HIP graph
// capture, tight serving loops) get their split-K planes, stream-K partial tiles and padded operand
// copies from this array instead of a hipMalloc'ed workspace.  Every GPU the library runs on holds
// its own copy at its own address until the process ends.  In host code the array's name is only a
// stand-in for the symbol: the device address comes from hipGetSymbolAddress(), once per device.
// The arrival counters in front come on top of the advertised size, so that a workspace of exactly that size fits: the
// planes of a split in four of 8192 x 512 are 64 MiB, and the same tile without a split takes twice as long.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = (size_t)HGEMM_STATIC_SCRATCH_BYTES;
constexpr size_t kCounterBytes = 64 * 1024;      // arrival counters of fused split-K plans: up to 16384 tiles
static __device__ __align__(256) unsigned char scratch[kCounterBytes + kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {nullptr};

// Device address of `scratch` on device `dev` (which must be the current device), or null.
void* scratch_ptr_for(int dev)
{
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

bool fast_path_ok(int64_t M, int64_t N, int64_t K, const hgemm_layouts_t& l)
{
    if (N % 8 || K % 8 || l.lda % 8 || l.ldb % 8 || l.ldc % 8) return false;
    // buffer offsets are 32-bit and bit 31 marks "out of range": keep every operand, including
    // the rows a padded tile may address, below 2 GiB
    const int64_t lim = (int64_t)1 << 31;
    const int64_t b_rows = (l.b == HGEMM_ROW_MAJOR) ? K : N;
    if ((M + 512) * l.lda * 2 >= lim || (b_rows + 512) * l.ldb * 2 >= lim || M * l.ldc * 2 >= ((int64_t)1 << 33)) return false;
    if ((N + 512) * K * 2 >= lim) return false;      // also the transposed copy of B, should a plan ask for one
    if (M >= (1 << 24) || N >= (1 << 24) || K >= (1 << 24)) return false;
    return true;
}

// Compute units of the current device, asked once per process.  Host-only callers on a machine
// without a GPU (the planner's helpers are usable there) get the MI355X figure.
int64_t cu_count()
{
    static const int64_t n = [] {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
            return (int64_t)prop.multiProcessorCount;
        (void)hipGetLastError();
        return (int64_t)256;
    }();
    return n;
}
constexpr double kCacheResidentBytes = 192.0 * 1024 * 1024;

// Last-resort rules, used only when neither the table nor the cost model yields a kernel this
// build holds.  They follow the trends of
// Section 6 (tile height/width grow with M/N; more stages for long K) with MI355X numbers:
// 256 CUs want >= 256 workgroups, so small problems take smaller tiles or split K.
Spec heuristic(int64_t M, int64_t N, int64_t K)
{
    Spec s;
    s.fam = FAM_MFMA;
    s.gm = 8;
    auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const int64_t CUS = cu_count();
    if (M <= 32) {
        s.bm = 32; s.bn = 128; s.bk = 64; s.wm = 1; s.wn = 4; s.st = 4;
    } else if (M <= 64) {
        s.bm = 64; s.bn = 128; s.bk = 64; s.wm = 2; s.wn = 2; s.st = 4;
    } else if (tiles(256, 256) >= CUS) {
        s.bm = 256; s.bn = 256; s.bk = 64; s.wm = 2; s.wn = 2; s.st = 2;
    } else if (tiles(128, 128) >= CUS || M * N >= (int64_t)2048 * 2048) {
        s.bm = 128; s.bn = 128; s.bk = 64; s.wm = 2; s.wn = 2; s.st = 4;
    } else {
        s.bm = 64; s.bn = 64; s.bk = 64; s.wm = 2; s.wn = 2; s.st = 4;
        if (M >= 128 && N >= 128 && tiles(128, 128) * 4 >= CUS) { s.bm = 128; s.bn = 128; }
    }
    // split K when the grid leaves most CUs idle and K is long enough to share
    const int64_t t = tiles(s.bm, s.bn);
    s.sk = 1;
    if (t < CUS && K >= 1024) {
        int64_t want = (2 * CUS + t - 1) / t;                 // aim at about two workgroups per CU
        int64_t max_by_k = K / (4 * s.bk);                    // at least four K-tiles per split
        s.sk = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(want, max_by_k), 64));
    }
    return s;
}

#include "dispatch_table.inc"
#include "dispatch_table_tn.inc"

// A table's rows in order of their shapes, with the logarithms that neighbour_choice compares: a call that plans (every
// hgemm_run_static does) looks its row up by bisection instead of walking a thousand rows.
struct TableIndex {
    struct Item { int64_t m, n, k; const char* spec; double lm, ln, lk; };
    std::vector<Item> items;
    TableIndex(const DispatchRow* rows, size_t count)
    {
        for (size_t i = 0; i < count; ++i) {
            const DispatchRow& r = rows[i];
            if (r.m > 0 && r.n > 0 && r.k > 0) items.push_back({r.m, r.n, r.k, r.spec, std::log2((double)r.m), std::log2((double)r.n), std::log2((double)r.k)});
        }
        std::stable_sort(items.begin(), items.end(), [](const Item& a, const Item& b) { return a.m != b.m ? a.m < b.m : a.n != b.n ? a.n < b.n : a.k < b.k; });
    }
    const char* find(int64_t M, int64_t N, int64_t K) const
    {
        auto it = std::lower_bound(items.begin(), items.end(), 0,
                                   [&](const Item& a, int) { return a.m != M ? a.m < M : a.n != N ? a.n < N : a.k < K; });
        return it != items.end() && it->m == M && it->n == N && it->k == K ? it->spec : nullptr;
    }
};
const TableIndex& table_index(bool b_col_major)
{
    static const TableIndex nn(kDispatchTable, sizeof(kDispatchTable) / sizeof(kDispatchTable[0]));
    static const TableIndex tn(kDispatchTableTN, sizeof(kDispatchTableTN) / sizeof(kDispatchTableTN[0]));
    return b_col_major ? tn : nn;
}

// The measured row for a shape: with column-major B the table tuned in that layout first, then (as for
// row-major B) the table tuned with row-major B, whose tile sizes and split factors carry over.
bool table_lookup(int64_t M, int64_t N, int64_t K, bool b_col_major, Spec* out)
{
    if (b_col_major) {
        const char* spec = table_index(true).find(M, N, K);
        if (spec && spec[0] != '\0' && parse_spec(spec, out)) return true;
    }
    // a row of the NN table serves a column-major B only if it names the large-tile family (the streaming
    // family decomposes the two layouts differently: slab and wave counts do not carry over)
    const char* spec = table_index(false).find(M, N, K);
    return spec && spec[0] != '\0' && parse_spec(spec, out) && !(b_col_major && out->fam != FAM_MFMA);
}

// ---------------------------------------------------------------------------
// Plan-time cost model for shapes the table does not hold.  Section 6 of the paper reads trends off
// its per-shape winners; here the dependence on (M, N, K) is an explicit model of one launch --
// matrix-core and copy time per K-tile, prologue/epilogue per workgroup, rounds over the compute
// units, whole-problem memory time, the second pass of split-K -- with constants fitted to measured
// times of all candidates on random shapes (plan_model.py holds the same formula and the fit).
// ---------------------------------------------------------------------------
struct PlanModel {
#define PLAN_MODEL_CONST(name, value) double name = value;
#include "plan_model.inc"
#undef PLAN_MODEL_CONST
};
const PlanModel kModel;

constexpr double kPadMinMacs = 1024.0 * 1024;     // below this many multiply-adds an unaligned problem stays on the generic kernel

// Split count finish_plan() will actually use: ranges are whole K-tiles, empty splits are dropped.
int64_t effective_splits(int64_t ktiles, int64_t sk)
{
    sk = std::min<int64_t>(sk, std::max<int64_t>(ktiles, 1));
    if (sk < 1) sk = 1;
    const int64_t per = (ktiles + sk - 1) / sk;
    return std::max<int64_t>(1, (ktiles + per - 1) / std::max<int64_t>(per, 1));
}

// Split factors worth considering for a configuration with `t` tiles and `ktiles` K-tiles.
struct SplitFactors {
    int n = 0, sk[12];
    const int* begin() const { return sk; }
    const int* end() const { return sk + n; }
};
SplitFactors split_candidates(int64_t t, int64_t ktiles)
{
    SplitFactors f;
    f.sk[f.n++] = 1;
    const int64_t kCUs = cu_count();
    if (t < 2 * kCUs) {
        for (int sk : {2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64}) {
            if (ktiles / sk < 2) break;
            if (t * sk > 8 * kCUs) break;
            f.sk[f.n++] = sk;
        }
    }
    return f;
}

// Tiles far taller or wider than the problem only waste matrix-core work.
bool tile_fits_problem(const MfmaEntry& e, int64_t M, int64_t N)
{
    if (e.bm >= 2 * M && e.bm > 32) return false;
    if (e.bn >= 2 * N && e.bn > 64) return false;
    return true;
}

// Predicted microseconds of one call (plain or split-K kernel, default tile order); big = predict_big(M, N, K).
double predict_big(int64_t M, int64_t N, int64_t K)
{
    const double flop = 2.0 * (double)M * (double)N * (double)K;
    return std::min(2.0, std::max(0.0, std::log10(std::max(flop, 1.0)) - 10.0)) / 2.0;
}
double predict_us(int64_t Mi, int64_t Ni, int64_t Ki, const MfmaEntry& e, int64_t ski, double big)
{
    const PlanModel& g = kModel;
    const int64_t kCUs = cu_count();
    const double M = (double)Mi, N = (double)Ni, K = (double)Ki;
    const int bm = e.bm, bn = e.bn, bk = e.bk, st = e.st, pf = e.pf, nw = e.wm * e.wn, tm = e.blocks_m, tn = e.blocks_n;
    const int64_t rows = (Mi + bm - 1) / bm;
    const double tiles = (double)(rows * ((Ni + bn - 1) / bn));
    const double kt = (double)((Ki + bk - 1) / bk);
    const double sk = (double)ski;
    const double occ = (double)e.resident;

    const double wgs = tiles * sk;
    const double kt_wg = std::ceil(kt / sk);
    const double w = std::ceil(wgs / (double)kCUs);
    const double co = std::min(occ, w);
    const double rounds = std::ceil(w / co);
    double t_mfma = 2.0 * bm * bn * bk / g.F * (1.0 + g.c1 * (double)(tm + tn) / (double)(tm * tn)) * (1.0 + g.cp * big);
    if (pf == 1) t_mfma *= g.q1;
    if (bm == 32) t_mfma *= g.m32;
    if (bk == 128) t_mfma *= g.k128; else if (bk == 32) t_mfma *= g.k32;
    const double stage = (double)(bm + bn) * bk * 2.0;
    const double bytes_in = 2.0 * (M * K + K * N);
    const double bytes_c = 2.0 * M * N;
    const double part = ski > 1 ? sk * M * N * 4.0 : 0.0;
    const bool resident = bytes_in + bytes_c < kCacheResidentBytes;
    const double miss = std::min(1.0, bytes_in / (wgs * kt_wg * stage));
    const double lat = g.L + miss * (resident ? 0.0 : g.Lh);
    double peak = g.BW * (nw == 2 ? g.a2 : nw == 8 ? g.a8 : nw == 16 ? g.a16 : 1.0);
    peak *= (bn == 64 ? g.b64 : bn == 256 ? g.b256 : 1.0);
    const double inflight = (double)std::max(st - 1, 1) * stage * co;
    const double bw = std::min(peak, inflight / lat) / co;
    const double t_copy = stage / bw;
    const double t_kt = std::max(t_mfma * co, t_copy) + g.ov * std::min(t_mfma * co, t_copy) + g.tk;        // ns
    const double pro = g.Tpro;
    const double epi = g.e0 + (ski > 1 ? bm * bn * 4.0 / g.BWp : bm * bn * 2.0 / g.BWepi) * 1e-3;
    const double cu_time = rounds * (kt_wg * t_kt * 1e-3 + pro + epi);
    const double tot_inflight = std::min(wgs, (double)kCUs * occ) * (double)std::max(st - 1, 1) * stage;
    const double bw_read = (resident && part + bytes_in + bytes_c < kCacheResidentBytes)
                               ? g.BWs
                               : std::min(g.BWh * (bn == 64 ? g.h64 : bn == 128 ? g.h128 : 1.0), tot_inflight / g.Lhb);
    const double writes = ski > 1 ? part : bytes_c;
    const double tiles_m = (double)rows;
    const double hbm_bytes = resident ? bytes_in : 2.0 * M * K + 2.0 * K * N * (1.0 + g.rr * (std::min(tiles_m, 8.0) - 1.0));
    const double t_main = std::max(cu_time, hbm_bytes / bw_read * 1e-3) + writes / (co <= 1.0 ? g.BWw1 : g.BWw2) * 1e-3;
    const double t_red = ski > 1 ? g.Tr0 + g.Tr1 * std::ceil(sk / 8.0) + (part + bytes_c) / g.BWr * 1e-3 : 0.0;
    return g.T0 + t_main + t_red;
}

// Predicted microseconds of one call of a skinny-family kernel: a launch floor, the chip-wide streaming
// time of B at a rate that grows with the number of workgroups in flight, the partial-plane traffic,
// and the reduction (a second launch, or the tail of the fused form).
struct SkinnyModel {
    // fitted (soft-L1 on log time, rms 0.095) to 107 measured (shape, slabs, fused) points of the register-transposing
    // kernel: M = 1, 16 on the C3 weights with every slab count, M = 1 .. 64 on weights of 112-448 MiB
    double t0 = 4.2;          // us: launch, first bytes and the waves' meeting at the end
    double bw = 6770.0;       // bytes/ns: chip-wide streaming rate with enough workgroups
    double wg_bw = 37.7;      // bytes/ns one workgroup sustains (its two steps of loads in flight)
    double round = 1.44;      // us of fill and drain per round of resident workgroups (3 per compute unit)
    double part_bw = 8750.0;  // bytes/ns for writing and re-reading fp32 planes
    double red2 = 1.93;       // us: second launch of the two-kernel reduction
    double red1 = 1.57;       // us: tail of the fused reduction
    double red1_per_mb = 5.0; // us more per MiB of planes when they are stored device-coherently
    double per_block = 0.28;  // relative cost of every further 16-row block of A (registers: fewer resident waves)
};
const SkinnyModel kSkinny;

double predict_skinny_us(int64_t M, int64_t N, int64_t K, int64_t sk, bool fused)
{
    const SkinnyModel& g = kSkinny;
    const double strips = (double)((N + kSkinnyCols - 1) / kSkinnyCols);
    const double wgs = strips * (double)sk;
    const double rate = std::min(g.bw, g.wg_bw * wgs);
    const double planes = sk > 1 ? (double)sk * M * N * 4.0 : 0.0;
    const double mblocks = M <= 16 ? 1.0 : M <= 32 ? 2.0 : 4.0;
    double t = g.t0 + 2.0 * (double)K * N / rate * 1e-3 * (1.0 + g.per_block * (mblocks - 1.0)) + std::ceil(wgs / (3.0 * (double)cu_count())) * g.round +
               2.0 * planes / g.part_bw * 1e-3;
    if (sk > 1) t += fused ? g.red1 + g.red1_per_mb * planes / 1048576.0 : g.red2;
    return t;
}

// The cheapest compiled configuration and split factor under the model.
// Split-K with the reduction fused into the kernel against the two-launch form, as fitted to skinny
// shapes (M = 1 and 16): the second launch (its dispatch gap and its own round trip) goes away, the planes are stored
// device-coherently (slower per byte), waited for and counted, and the last workgroup's re-read is a serial tail.  Too kind to the fused form, which takes
// 0.6-0.7 us longer than its two launches up to 32 rows (13 492 problems) and 1.4 us beyond (5138).  Beyond 32 rows the models pick two
// launches: 1706 problems for which they used to pick the fused form (and 699 of them now another split, or none) take 0.81 of their time from HBM and from the
// cache, 1 and 5 more than 1.03, and 0.66 planned, run and destroyed (no counters to clear).  Up to 32 rows, where the measured neighbours choose next, it stays: two launches 0.98 (237 of 5648 slower by more than 3 %).
double fused_delta_us(int64_t M, int64_t N, int64_t sk)
{
    const double planes_mib = (double)sk * (double)M * (double)N * 4.0 / 1048576.0;
    return -0.8 + 1.6 * planes_mib;
}

// Slab counts worth considering for the skinny family (distinct after rounding to whole steps of a
// four-wave workgroup, 64 rows).
std::vector<int> skinny_split_candidates(int64_t N, int64_t K)
{
    const int64_t ksteps = (K + 63) / 64, strips = (N + kSkinnyCols - 1) / kSkinnyCols;
    std::vector<int> out;
    int64_t last = 0;
    for (int sk : {1, 2, 4, 8, 16, 32, 64, 128}) {
        const int64_t eff = effective_splits(ksteps, sk);
        if (eff == last || strips * eff > 64 * cu_count()) continue;
        last = eff;
        out.push_back((int)eff);
    }
    return out;
}

// The streaming family's best slab count for a row-major B under its model, and the prediction.
double skinny_choice(int64_t M, int64_t N, int64_t K, Spec* out)
{
    double best = 1e300;
    for (int sk : skinny_split_candidates(N, K)) {
        for (int fr = 0; fr <= (sk > 1 ? 1 : 0); ++fr) {
            const double us = predict_skinny_us(M, N, K, sk, fr != 0);
            if (us < best) {
                best = us;
                Spec s;
                s.fam = FAM_SKINNY; s.sk = (int)sk; s.fr = fr;
                *out = s;
            }
        }
    }
    return best;
}

// A row-major B whose rows do not consist of whole aligned 16-byte chunks would have to be copied for the large-tile
// kernels; the streaming family reads it as it is.  Taken for M <= 32 always, and up to its 64 rows where B is 32 MiB or
// more and K 256: there the copy alone takes longer than the multiplication (40 x 32001 x 2048: copy and 64-row tiles 64 us,
// streamed 39), below that size the copy stays in the caches and the 64-row tiles are the faster half of the deal, and a
// shorter K is few steps of the stream per 128 columns of C (62 x 473671 x 48: streamed 83 us, with copies of A, B and C 68;
// of 220 such problems with K below 64 streamed 1.1 times, copied 0.64 times what three copies take; from K = 256 on 0.54 and 0.58).
bool streams_any_b(int64_t M, int64_t N, int64_t K, const hgemm_layouts_t& l)
{
    if (l.b != HGEMM_ROW_MAJOR || (N % 8 == 0 && l.ldb % 8 == 0) || N < 8 || M > kSkinnyMaxM) return false;
    if ((K + 512) * l.ldb * 2 >= ((int64_t)1 << 31)) return false;
    return M <= 32 || (K >= 256 && 2.0 * (double)K * (double)N >= 32.0 * 1048576.0);
}

// Few rows of A: the nearest of some four thousand measured problems (few_rows.inc; few_rows.py builds them from their timings and
// evaluates the choices) instead of the models' pick.  The models above are fitted to operands that the last-level cache holds (large
// tiles) or know one kernel of each family (streaming): on problems whose weights come from HBM their picks are 12 % slower than the
// fastest kernel, up to 1.6 times where 256-column tiles leave a third of the chip idle in their only round (4 x 23424 x 5120, column-major
// B: 63 us, in 128-column tiles 42).
// Distance = 0.3 |log2 ratio of M| + |log2 ratio of N| + |log2 ratio of K|, and a quarter more across 16384 and 32768 columns, where
// 64-column tiles begin another round; at most 0.3.  Rows of more than 32 rows of A are no neighbours: they fill the chip with
// 32-row tiles in pairs (24 x 18368 x 1088 took the kernel of 35 x 19208 x 1088, 13.2 us instead of 9.9).  A pick that is among the
// neighbour's fastest stays, one that needs no workspace is not traded for a split (as in phased_choice), and a split not for one of
// more planes unless these stay below the 2 MiB from which an allocation costs 60 us (and so far within the static scratch); nor one
// that needs more rounds of workgroups than the neighbour did, other than in proportion to its columns (within 5 %; 4 x 5480 x 12912: 258
// in two rounds 45 us, the model's pick 33); nor resident A for more than 16 rows and less than 16384 columns (99 such picks 1.06 times
// faster from HBM and 1.1 times slower from the cache).  Where a fused reduction was timed as the fastest of a problem, its two launches take
// 1.2 % longer from HBM and 0.5 % from the cache (692 problems), but it clears its counters in every new plan: 5 x 3840 x 3840 planned,
// run and destroyed 20.7 us, with counters 24.5.
// 4848 problems that the rows do not come from, a quarter of them of any sizes, in both states: 2498 choices differ from the models', 1.15 times
// faster from HBM and 1.13 from the cache; 131 and 185 of them are slower by more than 3 %, 40 and 54 by 10 %.  (Timed when a column-major B was
// loaded as operands; 983 of them go to strips_choice since.  The rows' streaming kernels of a column-major B have become faster since they were timed: where rows name
// one, 0.85 of the time of before on 84 problems, none slower; where they name a tile, one of them is the fastest for 211 of 1384.)
// Not for operands that would be copied: the choice between copies and direct_choice compares with the models' pick.
constexpr double kCheapAlloc = 2097152.0 - 65536.0;      // bytes of planes beside the counters below hipMalloc's 2 MiB step
struct FewRow { unsigned short m; unsigned n, k; signed char spec[5]; };
#include "few_rows.inc"
struct FewItem { float ln, lk, lm; int columns; };
// Rows stand in quarters of an octave of N and by K in each, so that a search looks at those within reach in both: some thirty of two
// thousand.  Nothing is allocated.
int columns_quarter(int64_t n)
{
    const int top = 63 - __builtin_clzll((unsigned long long)n);
    return 4 * top + (int)((n << 2 >> top) & 3);
}
template <size_t COUNT>
struct FewIndex {
    FewItem items[COUNT];
    unsigned short start[4 * 32 + 1] = {};       // of a quarter's rows
    explicit FewIndex(const FewRow (&rows)[COUNT])
    {
        for (size_t i = 0; i < COUNT; ++i) {
            items[i] = {std::log2((float)rows[i].n), std::log2((float)rows[i].k), std::log2((float)rows[i].m), std::min(3, (int)((rows[i].n + 16383) / 16384))};
            ++start[columns_quarter(rows[i].n) + 1];
        }
        for (size_t q = 1; q < std::size(start); ++q) start[q] += start[q - 1];
    }
};
struct FewKernels {
    Spec spec[std::size(kFewSpecs)];
    bool ok[std::size(kFewSpecs)];
    FewKernels()
    {
        for (size_t i = 0; i < std::size(kFewSpecs); ++i) ok[i] = parse_spec(kFewSpecs[i], &spec[i]) && (spec[i].fam != FAM_MFMA || find_entry(spec[i]));
    }
};
const FewRow* nearest_few_row(int64_t M, int64_t N, int64_t K, bool b_row_major)
{
    static const FewIndex nn(kFewRowsNN);
    static const FewIndex tn(kFewRowsTN);
    const FewItem* const items = b_row_major ? nn.items : tn.items;
    const unsigned short* const start = b_row_major ? nn.start : tn.start;
    const float lm = std::log2((float)M), ln = std::log2((float)N), lk = std::log2((float)K);
    const int columns = (int)std::min<int64_t>(3, (N + 16383) / 16384);
    float best = 0.3f;
    const FewItem* item = nullptr;
    for (int q = columns_quarter(std::max<int64_t>(1, (int64_t)((double)N * 0.8122))); q <= columns_quarter((int64_t)((double)N * 1.2312)); ++q) {      // 2^-0.3, 2^0.3
        const FewItem* const end = items + start[q + 1];
        for (const FewItem* r = std::lower_bound(items + start[q], end, lk - best, [](const FewItem& x, float v) { return x.lk < v; }); r != end && r->lk < lk + best; ++r) {
            const float d = 0.3f * std::fabs(lm - r->lm) + std::fabs(ln - r->ln) + std::fabs(lk - r->lk) + (columns != r->columns ? 0.25f : 0.f);
            if (d < best) { best = d; item = r; }
        }
    }
    return item ? (b_row_major ? kFewRowsNN : kFewRowsTN) + (item - items) : nullptr;
}
bool few_rows_choice(int64_t M, int64_t N, int64_t K, bool b_row_major, const Spec& model, Spec* out)
{
    static const FewKernels kernels;
    const FewRow* const row = nearest_few_row(M, N, K, b_row_major);
    if (!row) return false;
    auto rounds = [](const Spec& s, int64_t n) {
        const int64_t cus = cu_count();
        if (s.fam != FAM_MFMA) return s.ra ? ((n + 15) / 16 + cus - 1) / cus : 0;
        return ((n + s.bn - 1) / s.bn * s.sk + cus - 1) / cus;
    };
    bool found = false;
    for (const signed char i : row->spec) {
        if (i < 0) break;
        if (!kernels.ok[i]) continue;
        Spec s = kernels.spec[i];
        if (s.ra && ((M > 16 && N < 16384) || !skinny_strips(M <= 16 ? 1 : 2, K))) continue;
        const int64_t step = s.fam == FAM_MFMA ? s.bk : skinny_step(s, !b_row_major);
        s.sk = (int)effective_splits((K + step - 1) / step, s.sk);
        if (s.sk == 1) s.fr = 0;
        if (s.fam == model.fam && s.bm == model.bm && s.bn == model.bn && s.bk == model.bk && s.st == model.st && s.pf == model.pf && s.sk == model.sk &&
            s.fr == model.fr && s.wv == model.wv && s.nr == model.nr && s.ra == model.ra)
            return false;
        const bool small = (double)s.sk * (double)M * (double)((N + 7) / 8 * 8) * 4.0 <= kCheapAlloc;
        const bool fits = s.sk == 1 || (model.sk > 1 && (small || s.sk < model.sk || (s.sk == model.sk && s.fr <= model.fr)));
        const int64_t here = rounds(s, N), there = rounds(s, row->n);
        if (!found && fits && (here <= there || 20 * here * row->n <= 21 * there * N)) { *out = s; found = true; }
    }
    return found;
}

// Long column-major B and up to 16 rows, 1200 <= K <= 4096, from 16384 columns (four rounds of strips): A resident outright, the measured
// rows lie too far apart to reach all of it (1 x 32000 x 4096: 63.9 -> 43.7 us, 16 x 32000 x 4096 55.9 -> 47.1).  183 problems of the range:
// 1.22 times faster from HBM than the models' picks (4 slower by more than 3 %) and 1.14 than the best other kernel, 1.10 and 1.02 from the
// cache (32).  Not where 24000 to 32768 columns give 128-column tiles one full round and K is below 3200: there it is 1.04 times
// faster from HBM than the models' picks and 1.06 times slower from the cache (27 problems; 1 x 30144 x 2112 1.14).  Fewer columns leave
// the last round emptier, a longer K goes through the registers in two parts.
bool resident_a_range(int64_t M, int64_t N, int64_t K)
{
    return M <= 16 && N >= 16384 && K >= 1200 && K <= 4096 && (N < 24000 || N > 32768 || K >= 3200);
}
constexpr char kResidentA[] = "skinny,sk=1,wv=8,ra=1";

// Does hgemm_run_many put calls of this pick into one launch?  Strips leave such picks alone, and a plan that is only ever run call by call pays for it: strips
// would take 0.99 of its time at K 256-512, 0.92 to 768, 0.81 to 1024 and 0.7-0.85 beyond (1500 problems of up to 320 rows; from HBM and from the cache alike).
bool joins_launches(const Spec& s, int64_t M, int64_t N, int64_t K)
{
    return s.fam == FAM_MFMA && s.sk == 1 && !s.sm && !s.ps && !s.ph && !s.di && !s.tb && s.ac == 32 && s.mi == 32 &&
           2.0 * ((double)M * K + (double)K * N + (double)M * N) <= 8.0 * 1048576.0;
}

// More than 16 rows of A: strips of B times blocks of rows of A, by the same kernel, where one workgroup for every compute unit covers the problem.  The
// tile is the one with the fewest rows of A and B together, which is what a compute unit has to fetch of every k.  Tiles of the large
// family read each byte for more products, but want more of them than such problems have: their K is split, with planes and a second launch.
// Timed against the choices made without it on 37 488 random problems of 17 to 320 rows: 0.75 of their time from HBM (725 slower by more than 3 %, 245 by
// 10 %), 0.68 from the cache (312, 51), 0.37 planned, run once and freed; timed when tiles were dealt by strips, more than 32 to some XCDs.  Dealt evenly, on 4415 others
// on both sides of the limits, half of round sizes (`strips.py evaluate`): the 2803 that are taken 0.73 / 0.62 (54 and 9 slower from HBM, 5 and 1 from the
// cache; dealt by strips 0.76 / 0.66, 108 and 26, 10 and 4), the 1612 left 0.96 / 0.80.  Dealt by strips, from HBM / from the cache, by rows of A and B in a tile, and where it ends:
//  * 32: 0.59 / 0.57 at K 1024-2048, 0.66 / 0.60 to 3072, 0.74 / 0.65 to 4096, 0.85 / 0.70 to 6144, 1.0 / 0.75 to 8192, 1.25 / 0.9 beyond (a split leaves less
//    of K to each);
//  * 48: 0.70 / 0.65, 0.77 / 0.69, 0.83 / 0.75, then 0.98 / 0.77 to 4608, 1.05 / 0.75 to 5120; 64: 0.76 / 0.70, 0.82 / 0.69, 0.90 / 0.75, then 1.0 / 0.76;
//  * 80: 0.89 / 0.83, 0.87 / 0.78, to 3584 0.91 / 0.79, then 0.97 / 0.85; 96: 0.97 / 0.94, left out;
//  * fewer than twice as many columns as rows of A, where A's bytes are what HBM gives: 0.97 / 0.74 at 32 rows and K 4608-6144, 1.0 / 0.88 at 48 and K 3072-4608;
//  * K below 1024: such picks share launches, and a strip ends before its copies flow (80 rows, K below 1280: 1.1);
//  * 17 to 32 rows of A: tiles of 16 x 16 only (0.85 / 0.95 of strips of all rows); wider ones are level with those.
bool strip_tiles_choice(int64_t M, int64_t N, int64_t K, const Spec& pick, Spec* out)
{
    if (M > 320 || N % 8 || N < 64 || K < 1024 || K > 6144 || joins_launches(pick, M, N, K)) return false;
    const int64_t cus = cu_count();
    int best = 81, mr = 0, nr = 0;
    for (int a = 16; a <= 64 && a < M + 16; a += 16)
        for (int b = 16; b <= 64; b += 16) {
            if (((M + a - 1) / a) * ((N + b - 1) / b) > cus || a + b > best) continue;
            if (a + b == best && std::abs(a - b) >= std::abs(mr - nr)) continue;
            best = a + b; mr = a; nr = b;
        }
    if (!mr || (M <= 32 && (best > 32 || N % 16))) return false;
    const int64_t longest = 2 * M > N ? (best <= 32 ? 4608 : 3072) : best <= 32 ? 6144 : best <= 64 ? 4096 : 3584;
    if (K > longest || (best > 64 && K < 1280)) return false;
    *out = Spec();
    out->fam = FAM_SKINNY; out->mr = mr; out->nr = nr;
    return true;
}


// Column-major B, up to 32 rows of A and 12288 columns: one strip of 16, 32 or 48 rows of B for every compute unit, K split among its
// waves only, so that there are no planes and no second launch (skinny_tn_gemm_kernel).  Timed against the choices made without it,
// table rows among them, on 10 424 problems of 1 to 32 rows (widths of layers, and any multiples of 16 and 8): on the 5955 that this takes 0.83 of their
// time from HBM (109 slower by more than 3 %, 22 by 10 %) and 0.72 from the cache (92, 5); on 983 others (few_rows_check.jsonl.gz) 0.85 (39, 8) and 0.75 (33, 3).
// Where it ends, as time from HBM / from the cache against those choices:
//  * more than 12288 columns: strips of 64 rows 0.98-1.06 up to 16384 columns, several rounds of strips level beyond;
//  * K below 16 nr: a strip ends before its copies flow (nr = 32: K 256 1.0 / 0.95, 512 0.91 / 0.8; nr = 48: 512 0.98 / 0.9, 768 0.96 / 0.83);
//  * a long K on strips for few compute units, which a split spreads over more of them, sooner with more rows of A, whose bytes every
//    strip reads: up to 1024 columns K 8192 0.9 / 0.85 at M = 2, 1.3 / 0.9 at 16; 4097-5120 columns K 4096 0.92 / 0.83 at M = 4, 6144 1.16 /
//    0.85 at 16; 3073-4096 columns K 8192-16384 0.85-0.98 / 0.84 up to 16 rows, 1.13 / 0.87 at 24.  Near these limits strips are level from HBM, a third slower by more
//    than 3 % and a third faster, and 0.8 from the cache (161 problems);
//    `strips.py evaluate`, 5389 problems on both sides: the 3796 that are taken 0.80 / 0.71 (116 slower by more than 3 % and 28 by 10 % from HBM; 27 and 4), the 1593 left 1.20 / 0.93.
//  * picks whose calls share launches stay: 16 calls in one take what two take here;
//  * columns that are no whole strip of 16 keep the measured neighbours' kernels.
bool strips_choice(int64_t M, int64_t N, int64_t K, const Spec& pick, Spec* out)
{
    if (M > 16 && strip_tiles_choice(M, N, K, pick, out)) return true;
    if (M > 32 || N % 16 || N < 64 || N > 12288 || joins_launches(pick, M, N, K)) return false;
    const int64_t blocks = (N + 4095) / 4096;
    if (K < 256 * blocks) return false;
    const double filled = (double)N / (4096.0 * (double)blocks);
    const double work = (double)K * (double)(M + 8);
    if (filled <= 0.75 ? work > (filled <= 0.25 ? 100e3 : filled <= 0.625 ? 125e3 : 190e3) : M > 16 && blocks < 3 && work > 200e3) return false;
    *out = Spec();
    out->fam = FAM_SKINNY;
    if (blocks > 1) out->nr = (int)(16 * blocks);
    return true;
}

// The same for a row-major B, in strips of 32 columns: half a cache line of each of its rows, which HBM gives more slowly, so the range is shorter.  On 23 596
// random problems of 17 to 320 rows 0.80 of the time from HBM of the choices without it (84 slower by more than 3 %, 39 by 10 %), 0.65 from the cache
// (39, 13), 0.38 planned, run once and freed (timed when tiles were dealt by strips).  On 2196 others, half of round sizes (`strips.py evaluate`), the 1070 that
// are taken 0.82 / 0.61 (47 slower by more than 3 % and 17 by 10 % from HBM, 1 and none from the cache), the 1126 left 0.98 / 0.68.  Where it ends, from
// HBM / from the cache: tiles of 16 x 32 0.78 / 0.61 at K 1024-1536, 0.85 / 0.66 to 2048, 1.05 / 0.74 to 3072, 1.25 / 0.82 to 4096; of 32 x 32 0.9 / 0.75 to 2048, 1.0 / 0.78 to
// 3072, and level with strips of all rows up to 32; fewer than twice as many columns as rows 0.93 / 0.65 at K 1536-2048, a quarter of them slower; wider tiles 1.05 / 0.9.
// Rows of B a multiple of 1 KiB apart, whose half lines then come from fewer of the memory's channels, on at least 1536 columns and for up to 64 rows of A, which share
// less of them: 1.11 / 0.69 beyond K 1408, 79 of 125 slower from HBM by 10 % (20 x 2048 x 2048 7.8 / 6.4 -> 9.3 / 4.1 us); to 1408 0.92 / 0.65.
bool row_strip_tiles_choice(int64_t M, int64_t N, int64_t K, int64_t ldb, const Spec& pick, Spec* out)
{
    if (M <= 16 || M > 320 || N < 64 || K < 768 || K > 2048 || joins_launches(pick, M, N, K)) return false;
    const int64_t cus = cu_count(), strips = (N + 31) / 32;
    const int mr = (M + 15) / 16 * strips <= cus ? 16 : M > 32 && (M + 31) / 32 * strips <= cus ? 32 : 0;
    if (!mr || (2 * M > N && K > 1280)) return false;
    if (mr == 16 && M <= 64 && N >= 1536 && K > 1408 && ldb % 512 == 0) return false;
    *out = Spec();
    out->fam = FAM_SKINNY; out->mr = mr; out->nr = 32;
    return true;
}

bool evaluate_model(int64_t M, int64_t N, int64_t K, Spec* out, bool b_row_major, bool measured)
{
    double best = 1e300;
    bool found = false;
    if (b_row_major && M <= kSkinnyMaxM) {
        best = skinny_choice(M, N, K, out);
        found = best < 1e300;
    }
    // The large-tile model below was fitted to timings with the operands warm in the last-level cache wherever
    // they fit it, the streaming family's to operands streamed from HBM; the two are not comparable for a few
    // rows of A against weights that no cache holds (256 MiB and more).  Measured from HBM at M <= 32 the
    // streaming family is the faster one there (8 and 32 x 28672 x 8192: 81 / 94 us against 128 for the large-tile
    // pick; 8192 x 28672: 77 / 87 against 116; 4 x 16384 x 16384: 87 us, 77 % of the HBM rate); for weights of
    // 128-160 MiB the two families are level at M = 1 and the 32-row tiles ahead from M = 16 on (32 x 10240 x 8192:
    // 36 us against 51), so those stay with the model.
    if (found && M <= 32 && 2.0 * (double)K * (double)N >= 256.0 * 1048576.0) return true;
    const double big = predict_big(M, N, K);
    for (const MfmaEntry& e : registry()) {
        if (e.deep || e.mi != 32) continue;          // the cost model was not fitted to these kernels: the tuner's business
        if (!tile_fits_problem(e, M, N)) continue;
        const int64_t t = ((M + e.bm - 1) / e.bm) * ((N + e.bn - 1) / e.bn);
        const int64_t ktiles = (K + e.bk - 1) / e.bk;
        for (int sk0 : split_candidates(t, ktiles)) {
            const int64_t sk = effective_splits(ktiles, sk0);
            double us = predict_us(M, N, K, e, sk, big);
            const bool fuse = sk > 1 && M <= 32 && fused_delta_us(M, N, sk) < 0.0 && (int64_t)t * (int64_t)sizeof(int) <= (int64_t)kCounterBytes;
            if (fuse) us += fused_delta_us(M, N, sk);
            if (us < best) {
                best = us;
                found = true;
                Spec s;
                s.fam = FAM_MFMA; s.bm = e.bm; s.bn = e.bn; s.bk = e.bk; s.wm = e.wm; s.wn = e.wn; s.st = e.st; s.pf = e.pf;
                s.sk = (int)sk; s.gm = 8; s.fr = fuse ? 1 : 0;
                *out = s;
            }
        }
    }
    if (!found || !measured || M > 32) return found;
    Spec near;
    if (!b_row_major && resident_a_range(M, N, K) && parse_spec(kResidentA, &near)) *out = near;
    else if ((!b_row_major || 2.0 * (double)K * (double)N < 256.0 * 1048576.0) && few_rows_choice(M, N, K, b_row_major, *out, &near)) *out = near;
    return found;
}

// The model's pick.  Evaluating it takes some hundred candidates (10-20 us of host time, more than a small call takes on
// the device), and a program that plans on every call -- hgemm_run_static, the one-call Python wrapper -- comes back with a
// handful of shapes.  Each thread keeps its last picks, a function of its arguments alone, in a table of fixed
// size.
bool model_choice(int64_t M, int64_t N, int64_t K, Spec* out, bool b_row_major = true, bool measured = false)
{
    struct Pick { int64_t M, N, K; bool row, measured, found; Spec spec; };
    constexpr size_t kPicks = 64;
    static thread_local Pick picks[kPicks] = {};
    const uint64_t h = ((uint64_t)M * 0x9E3779B97F4A7C15ull ^ (uint64_t)N * 0xC2B2AE3D27D4EB4Full ^ (uint64_t)K * 0x165667B19E3779F9ull) + b_row_major + 2 * measured;
    Pick& p = picks[(h ^ (h >> 29)) % kPicks];
    if (p.M != M || p.N != N || p.K != K || p.row != b_row_major || p.measured != measured) {
        p.found = evaluate_model(M, N, K, &p.spec, b_row_major, measured);
        p.M = M; p.N = N; p.K = K; p.row = b_row_major; p.measured = measured;
    }
    if (p.found) *out = p.spec;
    return p.found;
}

// Large problems the table does not hold: the tuned choice of the nearest shape that it does hold.
// The cost model was fitted before the 16x16x32 kernels existed and never picks them, and on problems
// of many tiles a neighbour's winner carries over (25 off-table shapes of at least 10^11 flop: the
// neighbour's kernel is faster than the model's on 21, 4.7 % in the geometric mean) -- except where the
// neighbour's tile fills the last round of workgroups much worse than the model's pick does (3000 x
// 6144 x 4096: 288 tiles of 256 x 256 against 512 of 192 x 192, 18 % slower), which is what the
// comparison of the two fill ratios below rules out (with it: 20 of 136 shapes change, those 7.5 %
// faster in the geometric mean, none slower by more than 0.3 %).  Distance = sum over M, N, K of
// |log2 ratio|, at most 1.5.
double last_round_fill(const Spec& s, int64_t M, int64_t N)
{
    if (s.fam != FAM_MFMA || s.bm <= 0 || s.bn <= 0) return 0.0;
    const int64_t cus = cu_count();
    const int64_t t = ((M + s.bm - 1) / s.bm) * ((N + s.bn - 1) / s.bn) * std::max(1, s.sk);
    return (double)t / (double)(((t + cus - 1) / cus) * cus);
}

bool neighbour_choice(int64_t M, int64_t N, int64_t K, bool b_col_major, const Spec& model, Spec* out)
{
    if (2.0 * (double)M * (double)N * (double)K < 3e10 || std::min(M, N) < 512 || model.fam != FAM_MFMA) return false;
    auto lg = [](int64_t v) { return std::log2((double)std::max<int64_t>(v, 1)); };
    const double lm = lg(M), ln = lg(N), lk = lg(K);
    double best = 1.5;
    const TableIndex::Item* pick = nullptr;
    for (const TableIndex::Item& r : table_index(b_col_major).items) {
        if (r.spec[0] == '\0') continue;
        const double d = std::fabs(lm - r.lm) + std::fabs(ln - r.ln) + std::fabs(lk - r.lk);
        if (d <= best) { best = d; pick = &r; }
    }
    Spec near;
    if (!pick || !parse_spec(pick->spec, &near) || near.fam != FAM_MFMA || near.tb) return false;
    const MfmaEntry* e = find_entry(near);
    if (!e || !tile_fits_problem(*e, M, N)) return false;
    if (last_round_fill(near, M, N) < last_round_fill(model, M, N) - 0.1) return false;
    // Row by row (gm = 0) is a tuned shape's order where its columns of tiles are a multiple of the eight XCDs: each XCD then
    // keeps its columns of B in its own L2.  Otherwise it does not carry over (1297 x 5392 x 12336, 43 columns of 128 x 128
    // phased: 333 us, in bands of eight rows 217; 249 such problems: 7 % in the geometric mean from the cache, 4 % from memory).
    if (near.ph && near.gm == 0 && ((N + near.bn - 1) / near.bn) % 8 != 0) near.gm = 8;
    *out = near;
    return true;
}

int64_t up8(int64_t v) { return (v + 7) / 8 * 8; }
size_t up256(size_t b) { return (b + 255) / 256 * 256; }

// Can the matrix-core and streaming kernels run the plan's problem (a padded one with its copies made)?
bool kernels_can_run(const hgemm_plan_s* p)
{
    if (!p->padded) return fast_path_ok(p->M, p->N, p->K, p->lay);
    hgemm_layouts_t l = p->lay;
    if (p->any_b) l.ldb = up8(l.ldb);
    l.ldc = up8(p->N);                      // C is addressed in 64 bits, whatever its leading dimension
    return fast_path_ok(p->M, up8(p->N), p->K, l);
}

// Can the kernels that read operands through registers run the problem?  Any pitches and addresses; whole loads of 8 elements
// have to exist, and byte offsets, those of the K-tiles loaded ahead of the last one included, stay below 2^32.
bool direct_can_run(int64_t M, int64_t N, int64_t K, const hgemm_layouts_t& l)
{
    const int64_t lim = (int64_t)1 << 31, b_rows = l.b == HGEMM_ROW_MAJOR ? K : N;
    return M > 0 && N >= 8 && K >= 8 && M < (1 << 24) && N < (1 << 24) && K < (1 << 24) && (M + 512) * l.lda * 2 < lim && (b_rows + 512) * l.ldb * 2 < lim &&
           l.ldc < lim;
}

// Lays the padded copies of A and B, and the packed C, out in the workspace behind the counters and returns their bytes.
size_t place_copies(hgemm_plan_s* p)
{
    p->a_off = p->b_off = p->c_off = 0;
    if (!p->padded) return 0;
    const size_t M = (size_t)p->M, N = (size_t)up8(p->N), K = (size_t)p->K;
    p->b_off = p->copy_a || p->spare ? up256(M * K * 2) : 0;
    p->c_off = p->b_off + ((p->copy_b || p->spare) && !p->any_b ? up256(K * N * 2) : 0);
    return p->c_off + (p->copy_c ? up256(M * N * 2) : 0);
}

// hgemm_run_static accepts a problem by the scratch it would take with padded copies of all three operands: callers
// size their problems by that rule.  (A B that is streamed where it lies counts as copied; the planes of the slabs, which
// the large-tile kernels would not have needed, then go without counting, as long as what is really taken fits.)
bool over_static_scratch(const hgemm_plan_s* p, size_t ctr_bytes)
{
    if (!p->static_ws || !p->workspace_bytes) return false;
    const size_t taken = p->workspace_bytes - ctr_bytes;
    size_t counted = taken;
    if (p->padded && !p->copy_c) counted += up256((size_t)p->M * (size_t)up8(p->N) * 2);
    if (p->any_b) {
        counted += up256((size_t)p->K * (size_t)up8(p->N) * 2);
        if (p->spec.sk > 1) counted -= up256((size_t)p->spec.sk * (size_t)p->M * (size_t)up8(p->N) * sizeof(float));
    }
    return counted > kScratchBytes || taken > kScratchBytes;
}

// Gives the plan its workspace of p->workspace_bytes (static scratch or an allocation), points the
// partial-sum and counter arguments into it and clears the counters of an allocated one.
hgemm_status_t acquire_workspace(hgemm_plan_s* p, size_t partial_bytes, size_t ctr_bytes)
{
    GemmArgs& a = p->args;
    if (p->workspace_bytes && p->static_ws) {
        if (over_static_scratch(p, ctr_bytes)) { p->workspace_bytes = 0; return HGEMM_ERR_WORKSPACE; }
        p->workspace = scratch_ptr_for(p->device);
        if (!p->workspace) { p->workspace_bytes = 0; return HGEMM_ERR_LAUNCH; }
        if (partial_bytes) a.partial = (float*)((char*)p->workspace + p->partial_offset);
        if (ctr_bytes) a.counters = (int*)p->workspace;          // static arrays start out zero
    } else if (p->workspace_bytes) {
        if (hipMalloc(&p->workspace, p->workspace_bytes) != hipSuccess) {
            (void)hipGetLastError();
            p->workspace = nullptr;
            p->workspace_bytes = 0;
            return HGEMM_ERR_ALLOC;
        }
        if (partial_bytes) a.partial = (float*)((char*)p->workspace + p->partial_offset);
        if (ctr_bytes) {
            if (hipMemset(p->workspace, 0, ctr_bytes) != hipSuccess) {
                (void)hipGetLastError();
                (void)hipFree(p->workspace);
                p->workspace = nullptr;
                p->workspace_bytes = 0;
                return HGEMM_ERR_ALLOC;
            }
            a.counters = (int*)p->workspace;
        }
    }
    return HGEMM_OK;
}

// The main kernel of a large-tile plan.  Dynamic LDS beyond 64 KiB has to be requested for a kernel function, once per
// device: a bit per (device, configuration, kernel) keeps a call that plans from asking again.
bool select_kernel(hgemm_plan_s* p)
{
    const MfmaEntry* e = p->entry;
    const Spec& s = p->spec;
    const bool split = s.sk > 1;
    void (*const all[])(GemmArgs) = {e->plain, e->splitk, e->streamk, e->splitk_fused, e->persist, e->acc16, e->phased, e->phased_splitk, e->direct, e->direct_splitk, e->direct_fused};
    void (*const all_tn[])(GemmArgs) = {e->plain_tn, e->splitk_tn, e->streamk_tn, e->splitk_fused_tn, e->persist_tn, e->acc16_tn, e->phased_tn, e->phased_splitk_tn,
                                           e->direct_tn, e->direct_splitk_tn, e->direct_fused_tn};
    const int which = s.di ? (!split ? 8 : s.fr ? 10 : 9) : s.sm ? 2 : s.ps ? 4 : split && s.fr ? 3 : s.ph ? (split ? 7 : 6) : split ? 1 : s.ac == 16 ? 5 : 0;
    p->kernel = p->tn_kernel ? all_tn[which] : all[which];
    p->kernel_any = which != 0 ? p->kernel : p->tn_kernel ? e->plain_any_tn : e->plain_any;
    p->kernel_lds = s.ph ? e->phased_lds : s.di ? e->direct_lds : e->lds_bytes;
    if (!p->kernel) return false;
    if (p->kernel_lds <= 64 * 1024) return true;
    constexpr size_t kMaxEntries = 256;
    static std::atomic<unsigned> allowed[kMaxDevices][kMaxEntries] = {};
    const size_t idx = (size_t)(e - registry().data());
    const unsigned bit = 1u << (which + (p->tn_kernel ? 16 : 0));
    const bool keep = idx < kMaxEntries && p->device >= 0 && p->device < kMaxDevices;
    if (keep && (allowed[p->device][idx].load(std::memory_order_acquire) & bit)) return true;
    for (auto k : {p->kernel, p->kernel_any})
        if (hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, p->kernel_lds) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
    if (keep) allowed[p->device][idx].fetch_or(bit, std::memory_order_release);
    return true;
}

constexpr int kTnInstances = 4 * 3 * 4 * 2;
// More than 64 KiB of dynamic LDS: asked for once per kernel and device.
bool admit_skinny_lds(int dev, int instance, const SkinnyTnKernel& k)
{
    if (k.lds <= 64 * 1024) return true;
    static std::atomic<bool> allowed[kMaxDevices][kTnInstances + 2] = {};
    const bool keep = dev >= 0 && dev < kMaxDevices;
    if (keep && allowed[dev][instance].load(std::memory_order_acquire)) return true;
    if (hipFuncSetAttribute((const void*)k.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, k.lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (keep) allowed[dev][instance].store(true, std::memory_order_release);
    return true;
}

hgemm_status_t finish_plan(hgemm_plan_s* p)
{
    const int64_t M = p->M, N = p->N, K = p->K;
    Spec& s = p->spec;
    p->entry = nullptr;
    p->workspace = nullptr;
    p->workspace_bytes = 0;
    p->partial_offset = 0;
    p->tn_kernel = false;
    memset(&p->args, 0, sizeof p->args);
    p->skinny = nullptr;
    p->skinny_lds = 0;
    if (s.fam == FAM_GENERIC) return HGEMM_OK;
    if (s.fam == FAM_SKINNY) {
        // strips of columns x K slabs of whole steps; partial planes as for split-K
        if (!kernels_can_run(p) || M <= 0 || N <= 0 || K <= 0 || (M > kSkinnyMaxM && !s.mr)) return HGEMM_ERR_UNSUPPORTED;
        const bool tn = p->lay.b == HGEMM_COL_MAJOR;
        p->tn_kernel = tn;
        const int mb = s.mr ? s.mr / 16 : row_blocks_of_a(M);
        const int64_t row_blocks = s.mr ? (M + s.mr - 1) / s.mr : 1;
        const int64_t step = skinny_step(s, tn);
        const int64_t ksteps = (K + step - 1) / step;
        const int64_t sk = effective_splits(ksteps, s.sk);
        if (sk > 65535) return HGEMM_ERR_UNSUPPORTED;
        s.sk = (int)sk;
        if (sk == 1) s.fr = 0;
        if (row_blocks > 65535) return HGEMM_ERR_UNSUPPORTED;
        const bool nn_tiles = !tn && s.mr;
        // (the last copies reach up to 256 rows past B, of the 512 that fast_path_ok() keeps below 2 GiB)
        if (nn_tiles && (p->any_b || s.wv != 4 || s.nr != 32 || s.mr > 32)) return HGEMM_ERR_UNSUPPORTED;
        if (!tn && !nn_tiles && s.nr != 0 && s.nr != 16) return HGEMM_ERR_UNSUPPORTED;
        if ((!tn && !nn_tiles) || s.ra) s.nr = 0;
        if (p->any_b && s.wv != 4) return HGEMM_ERR_UNSUPPORTED;
        if (s.ra && (!tn || M > 32)) return HGEMM_ERR_UNSUPPORTED;
        // with A resident, one workgroup per compute unit (a multiple of the 8 XCDs) walks the strips
        const int64_t strips = s.ra ? std::max<int64_t>(8, cu_count() / 8 * 8) : (N + skinny_cols(s, tn || nn_tiles, M, N) - 1) / skinny_cols(s, tn || nn_tiles, M, N);
        if (s.fr && strips * (int64_t)sizeof(int) > (int64_t)kCounterBytes) return HGEMM_ERR_UNSUPPORTED;
        if ((tn && !s.ra) || nn_tiles) {
            const int rows = strip_rows(s, M, N);
            const SkinnyTnKernel k = nn_tiles ? skinny_tiles_kernel(mb) : skinny_tn_kernel(mb, s.fr != 0, s.wv, rows);
            const int instance = nn_tiles ? kTnInstances + mb - 1 : (((mb - 1) * 3 + s.wv / 8) * 4 + rows / 16 - 1) * 2 + s.fr;
            if (!k.kernel || !admit_skinny_lds(p->device, instance, k)) return HGEMM_ERR_UNSUPPORTED;
            p->skinny = k.kernel;
            p->skinny_lds = k.lds;
        } else {
            p->skinny = s.ra ? skinny_strips(mb, K) : p->any_b ? skinny_any_b_kernel(mb, s.fr != 0) : skinny_kernel(mb, s.fr != 0, s.wv);
        }
        if (!p->skinny) return HGEMM_ERR_UNSUPPORTED;
        GemmArgs& a = p->args;
        a.M = (int)M; a.N = (int)N; a.K = (int)K;
        a.lda = (int)p->lay.lda; a.ldb = (int)p->lay.ldb; a.ldc = (int)p->lay.ldc;
        a.tiles_m = (int)row_blocks; a.tiles_n = (int)strips;
        a.splits = (int)sk;
        a.k_per_split = s.ra ? (int)(ksteps * 32) : (int)(((ksteps + sk - 1) / sk) * step);      // of a wave, else of a slab
        a.b_rows = (int)(p->padded && !p->copy_b ? p->uK : K);
        // workspace: [counters] [padded copies of A and B (problems off the 16-byte grid)] [planes]
        const size_t pad_bytes = place_copies(p);
        const size_t partial_bytes = sk > 1 ? up256((size_t)sk * (size_t)M * (size_t)part_ld((int)N) * sizeof(float)) : 0;
        const size_t ctr_bytes = (s.fr || (p->static_ws && pad_bytes + partial_bytes > 0)) ? kCounterBytes : 0;
        p->a_off += ctr_bytes; p->b_off += ctr_bytes; p->c_off += ctr_bytes;
        p->bt_off = ctr_bytes + pad_bytes;
        p->partial_offset = ctr_bytes + pad_bytes;
        p->workspace_bytes = ctr_bytes + pad_bytes + partial_bytes;
        return acquire_workspace(p, partial_bytes, ctr_bytes);
    }
    const MfmaEntry* e = find_entry(s);
    if (!e) return HGEMM_ERR_UNSUPPORTED;
    if (s.di ? !e->direct || p->padded || !direct_can_run(M, N, K, p->lay) : !kernels_can_run(p)) return HGEMM_ERR_UNSUPPORTED;
    if (s.tb && p->lay.b != HGEMM_ROW_MAJOR) return HGEMM_ERR_UNSUPPORTED;
    p->tn_kernel = s.tb || p->lay.b == HGEMM_COL_MAJOR;
    p->entry = e;
    // deep-staged configurations exist for one full-K tile per workgroup only; the 16-bit accumulator for 32-wide blocks only
    if (e->deep && (s.sk > 1 || s.sm || s.ps || s.fr || s.ac == 16)) return HGEMM_ERR_UNSUPPORTED;
    if (s.ac == 16 && !e->acc16) return HGEMM_ERR_UNSUPPORTED;
    if (s.ph && !e->phased) return HGEMM_ERR_UNSUPPORTED;
    GemmArgs& a = p->args;
    a.M = (int)M; a.N = (int)N; a.K = (int)K;
    a.lda = (int)p->lay.lda; a.ldb = s.tb ? (int)K : (int)p->lay.ldb; a.ldc = (int)p->lay.ldc;
    a.tiles_m = (int)((M + e->bm - 1) / e->bm);
    a.tiles_n = (int)((N + e->bn - 1) / e->bn);
    if ((int64_t)a.tiles_m * a.tiles_n >= ((int64_t)1 << 24)) return HGEMM_ERR_UNSUPPORTED;      // tile_coords()
    // with a handful of tiles the order cannot matter: spare the kernel the arithmetic of the map
    a.swizzle = (int64_t)a.tiles_m * a.tiles_n <= 16 ? 0 : s.gm;
    set_tile_map(a);
    // split K into ranges that are multiples of BK; drop splits that would be empty
    int64_t ktiles = (K + e->bk - 1) / e->bk;
    const int64_t sk = effective_splits(ktiles, s.sk);
    const int64_t per = (ktiles + sk - 1) / sk;
    if (sk > 65535) return HGEMM_ERR_UNSUPPORTED;
    s.sk = (int)sk;
    if (sk == 1) s.fr = 0;                              // nothing to reduce
    if (s.ps) {
        if (!e->persist) return HGEMM_ERR_UNSUPPORTED;
        // persistent walking needs more tiles than compute units and a K long enough to keep the pipeline full
        if ((int64_t)a.tiles_m * a.tiles_n <= cu_count() || ktiles < e->st || sk > 1) s.ps = 0;
    }
    a.splits = (int)sk;
    a.k_per_split = (int)(per * e->bk);
    // stream-K geometry
    a.dp_tiles = a.tiles_m * a.tiles_n;
    a.sk_workers = 0;
    a.sk_iters_per_worker = 1;
    a.sk_total_iters = 0;
    if (s.sm) {
        const int64_t G = cu_count();
        const int64_t tiles = (int64_t)a.tiles_m * a.tiles_n;
        const int64_t dp = (tiles / G) * G;
        if (dp == tiles) {
            s.sm = 0;                                   // whole waves only: nothing to stream
        } else {
            const int64_t total = (tiles - dp) * ktiles;
            const int64_t ipw = (total + G - 1) / G;
            a.dp_tiles = (int)dp;
            a.sk_iters_per_worker = (int)ipw;
            a.sk_total_iters = (int)total;
            a.sk_workers = (int)((total + ipw - 1) / ipw);
        }
    }
    a.b_rows = (int)(p->padded && !p->copy_b ? p->uK : K);
    const size_t pad_bytes = place_copies(p);
    size_t bt_bytes = s.tb ? up256((size_t)N * (size_t)K * 2) : 0;
    size_t partial_bytes = sk > 1 ? (size_t)sk * (size_t)M * (size_t)part_ld((int)N) * sizeof(float) : 0;
    if (s.sm) partial_bytes = (size_t)2 * a.sk_workers * e->bm * e->bn * sizeof(float);
    partial_bytes = up256(partial_bytes);
    // fused split-K: one arrival counter per tile in front of everything else.  Counters are zero
    // whenever no launch is in flight (the last arriver resets its own), so their place is fixed:
    // the first kCounterBytes of the workspace, whatever the rest of it holds.
    // (In the static scratch every plan keeps clear of that region, so it stays zero for the fused ones.)
    const size_t ctr_bytes = (s.fr || (p->static_ws && pad_bytes + bt_bytes + partial_bytes > 0)) ? kCounterBytes : 0;
    if (s.fr && (size_t)a.tiles_m * a.tiles_n * sizeof(int) > kCounterBytes) return HGEMM_ERR_UNSUPPORTED;
    p->a_off += ctr_bytes; p->b_off += ctr_bytes; p->c_off += ctr_bytes;
    p->bt_off = ctr_bytes + pad_bytes;
    p->partial_offset = ctr_bytes + pad_bytes + bt_bytes;
    p->workspace_bytes = ctr_bytes + pad_bytes + bt_bytes + partial_bytes;
    if (!select_kernel(p)) return HGEMM_ERR_LAUNCH;
    return acquire_workspace(p, partial_bytes, ctr_bytes);
}

// Phased kernels on problems that the table does not hold.  The cost model above was fitted before they existed.  They
// have a model of their own, fitted (soft-L1 on log time, 850 timings on 240 random problems of at least 3e10 flop, operands
// rotated through 400 MB, rms 8-13 %): rounds of workgroups over the compute units, a K-tile the slower the larger the share
// of the chip that works, reads of A and B and the planes of a split at rates of their own.
struct PhasedTile { const char* spec; int bm, bn; double tk, fixed, busy, tail, bw, plane_bw, reduce, t0; };
constexpr PhasedTile kPhasedTiles[] = {
    {"mfma,bm=256,bn=256,bk=64,wm=2,wn=4,st=2,pf=1,sk=1,gm=8,mi=16,ph=1", 256, 256, 0.968, 8.218, 0.475, 1.0, 5.161, 3.986, 4.727, 0.3},
    {"mfma,bm=256,bn=128,bk=64,wm=2,wn=4,st=3,pf=1,sk=1,gm=8,mi=16,ph=1", 256, 128, 0.452, 4.214, 1.248, 1.0, 4.959, 3.337, 2.092, 4.0},
    {"mfma,bm=128,bn=256,bk=64,wm=2,wn=4,st=3,pf=1,sk=1,gm=8,mi=16,ph=1", 128, 256, 0.688, 3.758, 0.366, 0.995, 5.311, 3.612, 4.954, 1.557},
    {"mfma,bm=128,bn=128,bk=64,wm=2,wn=4,st=3,pf=1,sk=1,gm=8,ph=1", 128, 128, 0, 0, 0, 0, 0, 0, 0, 0},      // twins only (below)
};
double predict_phased_us(const PhasedTile& c, int64_t M, int64_t N, int64_t K, int64_t sk)
{
    const int64_t kt = (K + 63) / 64;
    sk = effective_splits(kt, sk);
    const double per = std::ceil((double)kt / (double)sk);
    const double wgs = (double)(((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * sk);
    const double rounds = wgs / (double)cu_count(), full = std::floor(rounds), part = rounds - full;
    auto round = [&](double share) { return per * c.tk * (1.0 + c.busy * share) + c.fixed; };
    const double cu = full > 0 ? full * round(1.0) + (part > 0 ? c.tail * round(part) : 0.0) : round(part);
    const double mem = 2.0 * ((double)M * K + (double)K * N + (double)M * N) / (c.bw * 1e6);
    const double main = std::pow(std::pow(cu, 6.0) + std::pow(mem, 6.0), 1.0 / 6.0);
    return c.t0 + main + (sk > 1 ? c.reduce + (double)sk * M * N * 4.0 / (c.plane_bw * 1e6) : 0.0);
}

bool same_tile(const Spec& s, const PhasedTile& c) { return s.fam == FAM_MFMA && s.bm == c.bm && s.bn == c.bn; }

// A phased kernel in the place of `pick` (the cost model's choice, or the nearest tuned shape's).
// From 3e10 flop: the phased tile and split with the smallest prediction, if that is below 0.95 of the pick's.  The cost
// model was fitted with operands in the last-level cache and is 13-16 % below measured times on problems of this size
// whose operands come from HBM: its predictions count 1.12 times.  A kernel that neither model knows stays.  A pick that
// needs no workspace is not traded for a split: a program that plans on every call would pay for the allocation
// (1024 x 2048 x 8192 through the one-call wrapper: 48 us, as a split 96).
// Below, or where no prediction is low enough: the phased schedule of the pick's own tile and split, if a split is long
// enough to pay for the longer prologue and epilogue (256 x 256: 128 of K, smaller tiles 384; 128 x 128 at K = 100: 10-20 %
// slower) and the rows of a row-major B start on cache lines where a unit is one line wide (BN = 128; 776 x 4056 x 2656:
// 6 % slower otherwise).
bool phased_choice(int64_t M, int64_t N, int64_t K, bool row_b, int64_t b_ld, const Spec& pick, Spec* out)
{
    if (pick.fam != FAM_MFMA || pick.ac != 32 || pick.tb) return false;
    if (pick.mi == 16 && !pick.ph && K / std::max(1, pick.sk) < 512) return false;
    const int most_sk = pick.sk > 1 || pick.sm ? 8 : 1;
    const double flop = 2.0 * (double)M * (double)N * (double)K;
    if (flop >= 3e10 && std::min(M, N) >= 96) {
        double limit = 0;                            // a kernel that neither model knows stays
        for (const PhasedTile& c : kPhasedTiles)
            if (pick.ph && c.tk > 0 && same_tile(pick, c)) limit = 0.95 * predict_phased_us(c, M, N, K, pick.sk);
        if (!pick.ph && !pick.sm && !pick.ps && pick.mi == 32) {
            const MfmaEntry* e = find_entry(pick);
            if (e && !e->deep)
                limit = 0.95 * 1.12 * predict_us(M, N, K, *e, effective_splits((K + pick.bk - 1) / pick.bk, pick.sk), predict_big(M, N, K));
        }
        const PhasedTile* best = nullptr;
        int best_sk = 1;
        for (const PhasedTile& c : kPhasedTiles) {
            if (c.tk <= 0 || c.bm >= 2 * M || c.bn >= 2 * N) continue;
            const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
            for (int sk : {1, 2, 3, 4, 6, 8}) {
                if (sk > most_sk || (sk > 1 && (tiles * sk > 640 || K / sk < 256))) break;
                if (2 * tiles * sk < cu_count()) continue;     // half the chip idle: outside what the model was fitted to choose
                const double us = predict_phased_us(c, M, N, K, sk);
                if (us < limit) { limit = us; best = &c; best_sk = sk; }
            }
        }
        if (best && parse_spec(best->spec, out)) {
            out->sk = best_sk;
            return true;
        }
    }
    if (pick.ph || pick.sm || pick.ps || pick.fr) return false;
    for (const PhasedTile& c : kPhasedTiles) {
        if (!same_tile(pick, c)) continue;
        const int64_t k_split = K / std::max(1, pick.sk);
        if (k_split < (c.bm == 256 && c.bn == 256 ? 128 : 384)) return false;
        if (row_b && c.bn == 128 && b_ld % 64 != 0) return false;
        if (!parse_spec(c.spec, out)) return false;
        out->sk = pick.sk;
        out->gm = pick.gm;
        return true;
    }
    return false;
}

// Problems off the 16-byte grid, read through registers where they lie.  Fitted (soft-L1 on log time; direct_model.py, which has the
// timings) to the four tiles and their splits on 588 random problems (M and N from 65 to 4200, K from 129; few rows against a long
// odd N among them), operands in the last-level cache.  late: what a K-tile takes longer when its operands come from HBM, loads being
// no more than two K-tiles ahead (90th percentile over the problems of 8 MB and more).
struct DirectTile { const char* spec; int bm, bn; double t0, wg, busy, flow, red2, red2_mib, red1, red1_mib, late; };
constexpr DirectTile kDirectTiles[] = {
#define DIRECT_TILE(...) {__VA_ARGS__},
#define DIRECT_COPIES(...)
#include "direct_model.inc"
#undef DIRECT_TILE
#undef DIRECT_COPIES
};
// Copies: a launch, the pick's prediction (warm and alone) this many times, and us for a MB read and written.
struct DirectCopies { double launch, kernel, mb; };
constexpr DirectCopies kDirectCopies =
#define DIRECT_TILE(...)
#define DIRECT_COPIES(...) {__VA_ARGS__};
#include "direct_model.inc"
#undef DIRECT_TILE
#undef DIRECT_COPIES
int64_t direct_ktiles(int64_t K, int64_t sk) { const int64_t kt = (K + 63) / 64; return ((kt + sk - 1) / sk + 1) / 2 * 2; }      // of a workgroup: whole pairs
double predict_direct_us(const DirectTile& c, int64_t M, int64_t N, int64_t K, int64_t sk, bool fused)
{
    sk = effective_splits((K + 63) / 64, sk);
    const double x = (double)(((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * sk) / (double)cu_count(), w = std::ceil(x);
    const double chain = c.busy * w, flow = c.flow * x;
    const double planes = (double)sk * M * N * 4.0 / 1048576.0;
    const double t = c.t0 + c.wg * w + (double)direct_ktiles(K, sk) * std::sqrt(std::sqrt(chain * chain * chain * chain + flow * flow * flow * flow));
    return sk == 1 ? t : t + (fused ? c.red1 + c.red1_mib * planes : c.red2 + c.red2_mib * planes);
}

// Predicted microseconds of one call of a specialisation, where a model knows it.
bool predict_spec_us(int64_t M, int64_t N, int64_t K, const Spec& s, double* us)
{
    if (s.fam == FAM_SKINNY) {
        if (M > kSkinnyMaxM || s.ra || s.mr) return false;         // fitted to kernels that stream slabs of K
        const int64_t eff = effective_splits((K + skinny_step(s) - 1) / skinny_step(s), s.sk);
        *us = predict_skinny_us(M, N, K, eff, s.fr != 0 && eff > 1);
        return true;
    }
    const MfmaEntry* own = s.fam == FAM_MFMA ? find_entry(s) : nullptr;
    if (!own || s.sm || s.tb || s.ps || s.ac == 16) return false;
    if (s.di) {
        for (const DirectTile& c : kDirectTiles)
            if (c.bm == s.bm && c.bn == s.bn) {
                *us = predict_direct_us(c, M, N, K, s.sk, s.fr != 0);
                return own->direct != nullptr;
            }
        return false;
    }
    if (s.ph) {
        // the cost model does not know the phased schedule: it counts like the best schedule of its tile that the model knows
        if (s.fr || !own->phased) return false;
        *us = 1e300;
        for (const MfmaEntry& e : registry()) {
            if (e.bm != s.bm || e.bn != s.bn || e.deep || e.mi != 32) continue;
            *us = std::min(*us, predict_us(M, N, K, e, effective_splits((K + e.bk - 1) / e.bk, s.sk), predict_big(M, N, K)));
        }
        return true;
    }
    const int64_t eff = effective_splits((K + s.bk - 1) / s.bk, s.sk);
    *us = predict_us(M, N, K, *own, eff, predict_big(M, N, K));
    if (s.fr && eff > 1) *us += fused_delta_us(M, N, eff);
    return true;
}

// True when device `dev` is a gfx950; the answer is kept per device (hipGetDeviceProperties is slow).
bool device_is_gfx950(int dev)
{
    static std::mutex m;
    static signed char known[kMaxDevices] = {0};       // 0 = not asked yet, 1 = yes, -1 = no
    if (dev < 0 || dev >= kMaxDevices) return false;
    std::lock_guard<std::mutex> lock(m);
    if (known[dev] == 0) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess) { (void)hipGetLastError(); return false; }
        known[dev] = strncmp(prop.gcnArchName, "gfx950", 6) == 0 ? 1 : -1;
    }
    return known[dev] == 1;
}

// Fills *p (caller's storage) with a runnable plan.  static_ws: the workspace is the device's static
// scratch array and nothing is allocated; otherwise the workspace is hipMalloc'ed and owned by the plan.
// The specialisation the planner tries first for an aligned problem of less than 2 GiB per operand, and where
// it comes from: the layout's dispatch table (packed leading dimensions only), else the cost model, whose pick a
// large problem trades for the kernel tuned for the nearest shape of the table (neighbour_choice), and either of them for a
// phased kernel (phased_choice).
// any_b: B is to be streamed where it lies (streams_any_b), which only the streaming family does.
// Returns the specialisations to try in order (a later one if the device or the workspace refuses an earlier one) and
// says where the first comes from.
// b_ld: the leading dimension of B as the kernels see it (l describes the packed problem of a padded one); copied: an operand is
// copied first, copy_b: B is.  A streaming row of the table is no pick for a column-major B that is copied first: it is worth reading B once, and
// direct_choice knows what to do with a pick of the large tiles.  96 such problems next to those rows: 1.9 times slower with the copies from HBM and 2.4
// from the cache than read in place (16 x 14336 x 4095 57 us, 31; 16 x 4096 x 4095 22, 14).  Copies of A only, or a C of odd rows, leave
// the rows the faster choice (0.93 of the large tiles' time from HBM, 0.85 from the cache).
struct Choices {
    const char* source;
    int n;
    Spec spec[3];
};
Choices choose_spec(int64_t M, int64_t N, int64_t K, const hgemm_layouts_t& l, int64_t b_ld, bool padded, bool copied, bool copy_b, bool any_b)
{
    Choices c{"table", 1, {}};
    const bool tn = l.b == HGEMM_COL_MAJOR;
    if (any_b && skinny_choice(M, N, K, &c.spec[0]) < 1e300) {
        c.source = "model";
        return c;
    }
    const bool packed = l.lda == K && l.ldc == N && l.ldb == (tn ? K : N);
    Spec model, near, phased;
    if (!packed || !table_lookup(M, N, K, tn, &c.spec[0]) || (tn && copy_b && c.spec[0].fam == FAM_SKINNY)) {
        c.source = "model";
        if (!model_choice(M, N, K, &model, !tn, !copied)) {
            model = heuristic(M, N, K);
            c.source = "rules";
        }
        c.n = 0;
        const bool neighbour = neighbour_choice(M, N, K, tn, model, &near);
        if (phased_choice(M, N, K, l.b == HGEMM_ROW_MAJOR, b_ld, neighbour ? near : model, &phased)) c.spec[c.n++] = phased;
        else if (neighbour) c.source = "neighbour";
        if (neighbour) c.spec[c.n++] = near;
        c.spec[c.n++] = model;
    } else if (c.spec[0].ph && c.spec[0].sk > 1) {
        c.spec[c.n] = c.spec[0];                  // where there is no room for the planes: the same tile without a split
        c.spec[c.n++].sk = 1;
    }
    Spec strips;
    if (!tn && !padded && strcmp(c.source, "table") && c.n < 3 && row_strip_tiles_choice(M, N, K, l.ldb, c.spec[0], &strips)) {
        for (int i = c.n++; i > 0; --i) c.spec[i] = c.spec[i - 1];
        c.spec[0] = strips;
    }
    if (tn && !padded && strcmp(c.source, "table") && c.n < 3 && strips_choice(M, N, K, c.spec[0], &strips)) {
        for (int i = c.n++; i > 0; --i) c.spec[i] = c.spec[i - 1];
        c.spec[0] = strips;
    }
    for (int i = 0; i < c.n; ++i)
        if (tn || padded) c.spec[i].tb = 0;       // B already has K contiguous / is copied once already
    return c;
}

// How hgemm_plan takes a problem: on the kernels that read aligned 16-byte chunks (`fast`), with packed zero-filled copies
// of those operands that cannot be read that way where they lie (`padded`), or neither.
struct Route {
    bool fast, padded, copy_a, copy_b, copy_c, any_b;
    int64_t N, K;                // the planner's view of the problem: rounded up to 8 where it is padded,
    hgemm_layouts_t lay;         // its operands packed
    int64_t lda, ldb, ldc;       // leading dimensions as the kernels see them
};
Route route(int64_t M, int64_t N, int64_t K, const hgemm_layouts_t& l)
{
    Route r{false, false, false, false, false, false, N, K, l, l.lda, l.ldb, l.ldc};
    if (M <= 0 || N <= 0 || K <= 0) return r;
    r.fast = fast_path_ok(M, N, K, l);
    // N, K or a leading dimension is not a multiple of 8.  Above a size where the one-thread-per-element kernel would
    // take longer than an extra launch, run the matrix-core kernels.
    if (r.fast || (double)M * (double)N * (double)K < kPadMinMacs) return r;
    const bool row_b = l.b == HGEMM_ROW_MAJOR;
    const int64_t Kp = up8(K), Np = up8(N);
    hgemm_layouts_t lp = l;
    lp.lda = Kp;
    lp.ldb = row_b ? Np : Kp;
    lp.ldc = Np;
    if (!fast_path_ok(M, Np, Kp, lp)) return r;
    // readable where it lies: rows of whole aligned chunks, and the kernels' offsets reach all of it
    hgemm_layouts_t la = lp, lb = lp;
    la.lda = l.lda;
    lb.ldb = l.ldb;
    r.copy_a = K % 8 != 0 || !fast_path_ok(M, Np, Kp, la);
    r.copy_b = (row_b ? N : K) % 8 != 0 || !fast_path_ok(M, Np, Kp, lb);
    r.any_b = r.copy_b && streams_any_b(M, N, K, l);
    if (r.any_b) r.copy_b = false;
    r.fast = r.padded = true;
    r.N = Np; r.K = Kp; r.lay = lp;
    r.lda = r.copy_a ? Kp : l.lda;
    r.ldb = r.copy_b ? lp.ldb : l.ldb;
    if (l.ldc >= ((int64_t)1 << 31)) {           // kernels have the pitch of C in 32 bits
        r.ldc = Np;
        r.copy_c = M > 1;
    }
    return r;
}

// A problem that would be copied: the kernels that read it where it lies instead?  `pick` is what the padded problem would run on;
// a phased or persistent pick stays, and so does a B that is streamed.  A copy costs a launch and the operand three times; reading through registers costs the
// matrix cores their even supply: 1000 x 1001 x 1003 11.1 -> 8.6 us, 500 x 501 x 503 7.4 -> 5.3, 70 x 3001 x 1001 11.3 -> 7.0, 2000 x 2001 x 2003
// 33 -> 29 (operands in the last-level cache), but 4100 x 4101 x 4103 183 -> 280.  Taken where its prediction is below 0.9 of the other way's (1.3
// times the prediction of the pick, which was fitted warm and alone, and 0.2 us a MB copied), below 0.75 for an unsplit K of 2560 and
// more, where it is the less certain one; and where it stays below with what operands from HBM add (in full from 16 MB on), by a tenth in
// more than one round of workgroups, by a twentieth with column-major B; 128 x 128 tiles up to one for every compute unit.  Two
// ranges keep their copies: a C of more than 4M elements with at most two K-tiles, where storing C takes most of the time
// (1980 x 13416 x 104 23 us, in place 33; 99 such problems 1.1 times slower), and a B beyond the cache that is not copied anyway, in more
// than one round of workgroups (53 x 53440 x 3213 64 us, in place 74).
// 6955 problems that the first condition takes, a third of them random and the others where it was in doubt: from HBM 1.30 times faster than the
// copies but 440 slower by more than 3 % and 222 by 10 % (up to 1.64 times), from the cache 1.39 times faster and 133 slower.
// Of the 5776 that all conditions leave, 59 are slower from HBM (8 by 10 %) and 8 from the cache; 1.36 and 1.44 times faster
// (`direct_model.py evaluate`).  Stricter ones cost more than they save: below 0.9 with the addition 11 are slower, but 667 more keep copies
// that are 1.13 times slower.
// A split whose planes pass the 2 MiB from which an allocation costs 60 us, where the copies stay below, is not considered (411 x 279 x 1277
// through the one-call wrapper 27 -> 60 us).
bool direct_choice(int64_t M, int64_t N, int64_t K, const hgemm_layouts_t& l, const Route& r, const Spec& pick, Spec* out)
{
    if (!r.padded || !(r.copy_a || r.copy_b) || r.any_b || pick.fam != FAM_MFMA || pick.ph || pick.ps || !direct_can_run(M, N, K, l) || 2.0 * (double)M * (double)N * (double)K > 4e10) return false;
    double other = 0;
    if (!predict_spec_us(M, r.N, r.K, pick, &other)) return false;
    const double moved = 4e-6 * ((r.copy_a ? (double)M * r.K : 0.0) + (r.copy_b ? (double)r.N * r.K : 0.0));      // MB read and written
    other = kDirectCopies.launch + kDirectCopies.kernel * other + kDirectCopies.mb * moved;
    // the workspace of the way with copies
    const double room = 2.0 * ((double)M * r.K + (double)r.N * r.K) + (pick.sk > 1 ? (double)pick.sk * (double)M * (double)r.N * 4.0 : 0.0);
    const DirectTile* best = nullptr;
    double best_us = 1e300;
    int best_sk = 1, best_fr = 0;
    const int64_t ktiles = (K + 63) / 64;
    for (const DirectTile& c : kDirectTiles) {
        const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
        if ((c.bm >= 2 * M && c.bm > 32) || (c.bn >= 2 * N && c.bn > 64) || (c.bm == 128 && tiles > cu_count())) continue;
        for (int sk : {1, 2, 3, 4, 6, 8, 12, 16}) {
            if (sk > 1 && (tiles * sk > 4 * cu_count() || ktiles / sk < 2 || tiles > cu_count())) break;
            const double planes = (double)effective_splits(ktiles, sk) * (double)M * (double)r.N * 4.0;
            if (sk > 1 && planes > kCheapAlloc && room <= kCheapAlloc) break;
            for (int fr = 0; fr < (sk > 1 && (double)sk * M * N * 4.0 <= 6.0 * 1048576.0 ? 2 : 1); ++fr) {
                const double us = predict_direct_us(c, M, N, K, sk, fr != 0);
                if (us < best_us) { best_us = us; best = &c; best_sk = sk; best_fr = fr; }
            }
        }
    }
    if (!best || ((double)M * (double)N > 4e6 && K <= 128)) return false;
    best_sk = (int)effective_splits(ktiles, best_sk);
    const double bytes = 2.0 * ((double)M * l.lda + (double)(l.b == HGEMM_ROW_MAJOR ? K : N) * l.ldb);
    const int64_t groups = ((M + best->bm - 1) / best->bm) * ((N + best->bn - 1) / best->bn) * best_sk;
    if (!r.copy_b && bytes > 128e6 && groups > cu_count()) return false;
    const double late = best->late * (double)direct_ktiles(K, best_sk) * std::min(1.0, bytes / 16e6);
    if (best_us >= (K >= 2560 && best_sk == 1 ? 0.75 : 0.9) * other) return false;
    if (best_us + late >= (groups > cu_count() ? 0.9 : l.b == HGEMM_ROW_MAJOR ? 1.0 : 0.95) * other || !parse_spec(best->spec, out)) return false;
    out->sk = best_sk;
    out->fr = best_fr;
    return true;
}

// hgemm_run_static refuses a problem whose padded copies, with the planes of a split, take more than the scratch; callers size
// their problems by that rule, so it stays one also for a problem that needs none of them any more.
bool copies_fit_static_scratch(int64_t M, const Route& r, const Choices& c)
{
    const size_t copies = up256((size_t)M * r.K * 2) + up256((size_t)r.K * r.N * 2) + up256((size_t)M * r.N * 2);
    for (int i = 0; i < c.n; ++i)
        if (copies + (c.spec[i].sk > 1 ? up256((size_t)c.spec[i].sk * M * r.N * sizeof(float)) : 0) <= kScratchBytes) return true;
    return false;
}

hgemm_status_t init_blocked(hgemm_plan_s* p);

hgemm_status_t init_plan(hgemm_plan_s* p, int64_t M, int64_t N, int64_t K, const hgemm_layouts_t* layouts, const char* spec_text,
                         bool static_ws)
{
    if (M < 0 || N < 0 || K < 0) return HGEMM_ERR_INVALID_ARG;
    hgemm_layouts_t l;
    if (layouts) {
        l = *layouts;
    } else {
        l.a = l.b = l.c = HGEMM_ROW_MAJOR;
        l.lda = l.ldb = l.ldc = 0;
    }
    if ((l.a != HGEMM_ROW_MAJOR && l.a != HGEMM_COL_MAJOR) || (l.b != HGEMM_ROW_MAJOR && l.b != HGEMM_COL_MAJOR) ||
        (l.c != HGEMM_ROW_MAJOR && l.c != HGEMM_COL_MAJOR))
        return HGEMM_ERR_INVALID_ARG;
    if (l.a != HGEMM_ROW_MAJOR || l.c != HGEMM_ROW_MAJOR) return HGEMM_ERR_UNSUPPORTED;
    if (l.lda < 0 || l.ldb < 0 || l.ldc < 0) return HGEMM_ERR_INVALID_ARG;
    if (l.lda == 0) l.lda = K;
    if (l.ldb == 0) l.ldb = (l.b == HGEMM_ROW_MAJOR) ? N : K;
    if (l.ldc == 0) l.ldc = N;
    if (l.lda < K || l.ldc < N || l.ldb < ((l.b == HGEMM_ROW_MAJOR) ? N : K)) return HGEMM_ERR_INVALID_ARG;

    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return HGEMM_ERR_ARCH; }
    if (!device_is_gfx950(dev)) return HGEMM_ERR_ARCH;

    p->M = M; p->N = N; p->K = K; p->lay = l; p->device = dev;
    p->padded = false;
    p->static_ws = static_ws;
    p->copy_a = p->copy_b = p->copy_c = p->any_b = false;
    p->spare = true;
    p->planned = spec_text == nullptr;
    p->uN = N; p->uK = K; p->ulay = l;
    p->a_off = p->b_off = p->c_off = p->bt_off = 0;

    hgemm_status_t st;
    if (spec_text) {
        if (!parse_spec(spec_text, &p->spec)) return HGEMM_ERR_INVALID_ARG;
        st = finish_plan(p);
    } else {
        const Route r = route(M, N, K, l);
        const bool fast = r.fast;
        if (r.padded) {
            p->padded = true;
            p->copy_a = r.copy_a; p->copy_b = r.copy_b; p->copy_c = r.copy_c; p->any_b = r.any_b;
            p->K = r.K;
            p->lay.lda = r.lda; p->lay.ldb = r.ldb; p->lay.ldc = r.ldc;
            N = r.N; K = r.K; l = r.lay;
        }
        const bool dims_aligned = !(N % 8 || K % 8 || l.lda % 8 || l.ldb % 8 || l.ldc % 8) && M < (1 << 24) && N < (1 << 24) && K < (1 << 24);
        if (!fast && !static_ws && M > 0 && N > 0 && K > 0 && dims_aligned && init_blocked(p) == HGEMM_OK) return HGEMM_OK;
        if (!fast) {
            p->spec = Spec();
            st = finish_plan(p);
        } else {
            const Choices c = choose_spec(M, N, K, l, r.ldb, p->padded, r.copy_a || r.copy_b, r.copy_b, p->any_b);
            Spec direct;
            if (direct_choice(M, p->uN, p->uK, p->ulay, r, c.spec[0], &direct) && (!static_ws || copies_fit_static_scratch(M, r, c))) {
                const hgemm_plan_s padded = *p;
                p->padded = p->copy_a = p->copy_b = p->copy_c = p->any_b = false;
                p->K = p->uK;
                p->lay = p->ulay;
                p->spec = direct;
                if (finish_plan(p) == HGEMM_OK) return HGEMM_OK;
                *p = padded;                               // no memory for planes, say: the other way
            }
            for (const bool spare : {true, false}) {       // no memory: once more without the room that only misaligned calls use
                p->spare = spare;
                for (int i = 0; i < c.n; ++i) {
                    p->spec = c.spec[i];
                    st = finish_plan(p);
                    if (st == HGEMM_OK) return HGEMM_OK;
                }
                if (st != HGEMM_ERR_ALLOC || !p->padded) break;
            }
            if (st == HGEMM_ERR_UNSUPPORTED && p->any_b) {     // not the streaming family after all: B is copied
                p->any_b = false;
                p->copy_b = true;
                p->lay.ldb = l.ldb;
            }
            if (st == HGEMM_ERR_UNSUPPORTED) {
                // a table row naming a kernel this build lacks, or a row of the NN table, consulted for a
                // column-major B, that names the streaming family (row-major B only): the cost model decides
                if (!model_choice(M, N, K, &p->spec, l.b == HGEMM_ROW_MAJOR)) p->spec = heuristic(M, N, K);
                if (l.b == HGEMM_COL_MAJOR || p->padded) p->spec.tb = 0;
                st = finish_plan(p);
                if (st == HGEMM_ERR_UNSUPPORTED) {
                    p->spec = heuristic(M, N, K);
                    st = finish_plan(p);
                }
            }
            if (st != HGEMM_OK && st != HGEMM_ERR_WORKSPACE && p->padded) {   // e.g. no memory for the padded copies: the generic kernel needs none
                p->padded = p->copy_a = p->copy_b = p->copy_c = p->any_b = false;
                p->N = p->uN; p->K = p->uK; p->lay = p->ulay;
                p->spec = Spec();
                st = finish_plan(p);
            }
        }
    }
    return st;
}

void destroy_blocks(hgemm_plan_s* p)
{
    for (auto& row : p->sub)
        for (hgemm_plan_s*& q : row) {
            if (!q) continue;
            if (q->workspace && !q->static_ws && hipFree(q->workspace) != hipSuccess) (void)hipGetLastError();
            delete q;
            q = nullptr;
        }
    p->blocked = false;
}

// Plans a problem whose dimensions are aligned but whose operands reach 2 GiB as a grid of blocks (see
// hgemm_plan_s).  On failure the plan is left as it was, for the generic kernel.
// Block sizes for a problem whose dimensions are aligned but whose operands reach 2 GiB: rows per block of A and
// C, columns per panel of B and C (equal sizes, multiples of 256), whether a row-major B has to go through a
// transposed copy, and the layouts the blocks are planned for.  False when no such split exists.
bool block_sizes(int64_t M, int64_t N, int64_t K, const hgemm_layouts_t& l, int64_t* rows, int64_t* cols, bool* transposed, hgemm_layouts_t* block_lay)
{
    const int64_t lim = (int64_t)1 << 31;
    auto down256 = [](int64_t v) { return v / 256 * 256; };
    int64_t bm = std::min<int64_t>(M, std::min(down256((lim - 1) / (l.lda * 2) - 512), down256((((int64_t)1 << 33) - 1) / (l.ldc * 2))));
    if (bm <= 0) return false;
    hgemm_layouts_t sl = l;
    // can the matrix-core kernels address B as it lies?  (asked of a block of 256 rows)
    bool bt = false;
    if (l.b == HGEMM_ROW_MAJOR && !fast_path_ok(std::min<int64_t>(bm, 256), N, K, l)) {
        if ((K + 63) / 64 > 65535) return false;          // grid of the transposing copy
        bt = true;
        sl.b = HGEMM_COL_MAJOR;
        sl.ldb = K;
    }
    int64_t bn = N;
    if (sl.b == HGEMM_COL_MAJOR) {
        bn = std::min<int64_t>(N, down256((lim - 1) / (sl.ldb * 2) - 512));
        if (bn <= 0) return false;
    }
    // blocks of equal size (a multiple of 256) rather than full ones and a sliver
    auto even = [](int64_t total, int64_t most) {
        const int64_t parts = (total + most - 1) / most;
        return std::min(most, ((total + parts - 1) / parts + 255) / 256 * 256);
    };
    if (bm < M) bm = even(M, bm);
    if (bn < N) bn = even(N, bn);
    if (!fast_path_ok(bm, bn, K, sl)) return false;
    *rows = bm;
    *cols = bn;
    *transposed = bt;
    *block_lay = sl;
    return true;
}

hgemm_status_t init_blocked(hgemm_plan_s* p)
{
    const int64_t M = p->M, N = p->N, K = p->K;
    int64_t bm = 0, bn = 0;
    bool bt = false;
    hgemm_layouts_t sl;
    if (!block_sizes(M, N, K, p->lay, &bm, &bn, &bt, &sl)) return HGEMM_ERR_UNSUPPORTED;
    p->blocked_bt = bt;
    p->block_m = bm;
    p->block_n = bn;
    p->block_lay = sl;
    const int64_t rows[2] = {M >= bm ? bm : 0, M % bm}, cols[2] = {N >= bn ? bn : 0, N % bn};
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
            if (rows[i] == 0 || cols[j] == 0) continue;
            hgemm_plan_s* q = new (std::nothrow) hgemm_plan_s();
            hgemm_status_t st = q ? init_plan(q, rows[i], cols[j], K, &sl, nullptr, false) : HGEMM_ERR_ALLOC;
            if (st == HGEMM_OK && q->blocked) st = HGEMM_ERR_UNSUPPORTED;
            if (st != HGEMM_OK) {
                if (q) {
                    destroy_blocks(q);
                    if (q->workspace && hipFree(q->workspace) != hipSuccess) (void)hipGetLastError();
                    delete q;
                }
                destroy_blocks(p);
                return st;
            }
            p->sub[i][j] = q;
        }
    p->spec = Spec();
    p->entry = nullptr;
    p->skinny = nullptr;
    p->workspace = nullptr;
    p->workspace_bytes = 0;
    if (bt) {
        const size_t bytes = (size_t)N * (size_t)K * 2;
        if (hipMalloc(&p->workspace, bytes) != hipSuccess) {
            (void)hipGetLastError();
            p->workspace = nullptr;
            destroy_blocks(p);
            return HGEMM_ERR_ALLOC;
        }
        p->workspace_bytes = bytes;
    }
    p->blocked = true;
    return HGEMM_OK;
}

hgemm_status_t make_plan(hgemm_plan_t* out, int64_t M, int64_t N, int64_t K, const hgemm_layouts_t* layouts,
                         const char* spec_text)
{
    if (!out) return HGEMM_ERR_INVALID_ARG;
    hgemm_plan_s* p = new (std::nothrow) hgemm_plan_s();
    if (!p) return HGEMM_ERR_ALLOC;
    const hgemm_status_t st = init_plan(p, M, N, K, layouts, spec_text, false);
    if (st != HGEMM_OK) { delete p; return st; }
    *out = p;
    return HGEMM_OK;
}

}  // namespace

extern "C" {

hgemm_status_t hgemm_plan(hgemm_plan_t* out, int64_t M, int64_t N, int64_t K, const hgemm_layouts_t* layouts)
{
    return make_plan(out, M, N, K, layouts, nullptr);
}

hgemm_status_t hgemm_plan_override(hgemm_plan_t* out, int64_t M, int64_t N, int64_t K, const hgemm_layouts_t* layouts,
                                   const char* spec)
{
    if (!spec) return HGEMM_ERR_INVALID_ARG;
    return make_plan(out, M, N, K, layouts, spec);
}

hgemm_status_t hgemm_plan_choice(int64_t M, int64_t N, int64_t K, const hgemm_layouts_t* layouts, char* buf, size_t n)
{
    if (!buf || n == 0 || M < 0 || N < 0 || K < 0) return HGEMM_ERR_INVALID_ARG;
    hgemm_layouts_t l;
    if (layouts) l = *layouts; else { l.a = l.b = l.c = HGEMM_ROW_MAJOR; l.lda = l.ldb = l.ldc = 0; }
    if ((l.b != HGEMM_ROW_MAJOR && l.b != HGEMM_COL_MAJOR) || l.lda < 0 || l.ldb < 0 || l.ldc < 0) return HGEMM_ERR_INVALID_ARG;
    if (l.a != HGEMM_ROW_MAJOR || l.c != HGEMM_ROW_MAJOR) return HGEMM_ERR_UNSUPPORTED;
    if (l.lda == 0) l.lda = K;
    if (l.ldb == 0) l.ldb = (l.b == HGEMM_ROW_MAJOR) ? N : K;
    if (l.ldc == 0) l.ldc = N;
    if (l.lda < K || l.ldc < N || l.ldb < ((l.b == HGEMM_ROW_MAJOR) ? N : K)) return HGEMM_ERR_INVALID_ARG;
    std::string out;
    const bool nonempty = M > 0 && N > 0 && K > 0;
    const Route r = route(M, N, K, l);
    const bool fast = r.fast;
    const int64_t uN = N, uK = K;
    const hgemm_layouts_t ul = l;
    N = r.N; K = r.K; l = r.lay;
    int64_t rows = 0, cols = 0;
    bool bt = false;
    hgemm_layouts_t bl;
    const bool dims_aligned = !(N % 8 || K % 8 || l.lda % 8 || l.ldb % 8 || l.ldc % 8) && M < (1 << 24) && N < (1 << 24) && K < (1 << 24);
    if (!nonempty) {
        out = "empty";
    } else if (!fast && dims_aligned && block_sizes(M, N, K, l, &rows, &cols, &bt, &bl)) {
        char head[96];
        snprintf(head, sizeof head, "blocks,rows=%lld,cols=%lld%s", (long long)rows, (long long)cols, bt ? ",bt=1" : "");
        out = head;
    } else if (!fast) {
        out = "generic";
    } else {
        const Choices c = choose_spec(M, N, K, l, r.ldb, r.padded, r.copy_a || r.copy_b, r.copy_b, r.any_b);
        Spec direct;
        if (direct_choice(M, uN, uK, ul, r, c.spec[0], &direct)) out = "model: " + spec_to_string(direct) + ",pad=1";
        else out = std::string(c.source) + ": " + spec_to_string(c.spec[0]) + (r.padded ? ",pad=1" : "");
    }
    if (out.size() + 1 > n) { buf[0] = '\0'; return HGEMM_ERR_INVALID_ARG; }
    memcpy(buf, out.c_str(), out.size() + 1);
    return HGEMM_OK;
}

static dim3 skinny_grid(const GemmArgs& a) { return dim3((unsigned)(a.tiles_n * a.tiles_m), (unsigned)a.splits); }

static hgemm_status_t run_plan(const hgemm_plan_s* plan, const void* A, const void* B, void* C, void* hip_stream)
{
    const int64_t M = plan->M, N = plan->N, K = plan->K;
    if (M == 0 || N == 0) return HGEMM_OK;
    if (!C) return HGEMM_ERR_INVALID_ARG;
    hipStream_t stream = (hipStream_t)hip_stream;
    if (K == 0) {
        const int wide = (((uintptr_t)C & 15) == 0 && plan->lay.ldc % 8 == 0) ? 1 : 0;
        hipLaunchKernelGGL(zero_c_kernel, dim3((unsigned)((N + 2047) / 2048), (unsigned)std::min<int64_t>(M, 16384)), dim3(256), 0, stream,
                           (_Float16*)C, M, N, plan->lay.ldc, wide);
        return hipGetLastError() == hipSuccess ? HGEMM_OK : HGEMM_ERR_LAUNCH;
    }
    if (!A || !B) return HGEMM_ERR_INVALID_ARG;

    if (plan->blocked) {
        const _Float16* Bp = (const _Float16*)B;
        if (plan->blocked_bt) {
            hipLaunchKernelGGL(transpose_kernel, dim3((unsigned)((N + 63) / 64), (unsigned)((K + 63) / 64)), dim3(256), 0, stream,
                               (const _Float16*)B, (_Float16*)plan->workspace, (int)K, (int)N, (int)plan->lay.ldb);
            if (hipGetLastError() != hipSuccess) return HGEMM_ERR_LAUNCH;
            Bp = (const _Float16*)plan->workspace;
        }
        const bool panels = plan->block_lay.b == HGEMM_COL_MAJOR;          // else every block takes all of B
        for (int64_t m0 = 0; m0 < M; m0 += plan->block_m)
            for (int64_t n0 = 0; n0 < N; n0 += plan->block_n) {
                const hgemm_plan_s* q = plan->sub[M - m0 < plan->block_m ? 1 : 0][N - n0 < plan->block_n ? 1 : 0];
                if (!q) return HGEMM_ERR_INVALID_ARG;
                const hgemm_status_t st = run_plan(q, (const _Float16*)A + m0 * plan->lay.lda, panels ? Bp + n0 * plan->block_lay.ldb : Bp,
                                                   (_Float16*)C + m0 * plan->lay.ldc + n0, hip_stream);
                if (st != HGEMM_OK) return st;
            }
        return HGEMM_OK;
    }

    // operands as the kernels see them: the caller's, or the padded copies made here
    int64_t lda = plan->lay.lda, ldb = plan->lay.ldb, b_rows = plan->args.b_rows;
    const bool row_b = plan->lay.b == HGEMM_ROW_MAJOR;
    if (plan->padded && plan->spec.fam != FAM_GENERIC) {
        const bool copy_a = plan->copy_a || (plan->spare && ((uintptr_t)A & 15));
        const bool copy_b = plan->copy_b || (plan->spare && ((uintptr_t)B & 15) && !plan->any_b);
        if (copy_a || copy_b) {
            char* ws = (char*)plan->workspace;
            const int64_t Np = up8(N);
            auto job = [](const void* src, int64_t src_ld, int64_t rows, int64_t cols, void* dst, int64_t dst_rows, int64_t dst_cols) {
                return PadCopy{(const _Float16*)src, (_Float16*)dst, src_ld, (unsigned)rows, (unsigned)cols, (unsigned)(dst_cols / 8),
                               (unsigned)(dst_rows * (dst_cols / 8))};
            };
            PadCopy ca{}, cb{};
            if (copy_a) ca = job(A, plan->ulay.lda, M, plan->uK, ws + plan->a_off, M, K);
            if (copy_b) cb = row_b ? job(B, plan->ulay.ldb, plan->uK, N, ws + plan->b_off, K, Np) : job(B, plan->ulay.ldb, N, plan->uK, ws + plan->b_off, N, K);
            constexpr unsigned per = 256 * kPadChunks;
            const unsigned blocks_a = (ca.total + per - 1) / per, blocks_b = (cb.total + per - 1) / per;
            hipLaunchKernelGGL(pad_copy_kernel, dim3(blocks_a + blocks_b), dim3(256), 0, stream, ca, cb, blocks_a);
            if (hipGetLastError() != hipSuccess) return HGEMM_ERR_LAUNCH;
            if (copy_a) { A = ws + plan->a_off; lda = K; }
            if (copy_b) { B = ws + plan->b_off; ldb = row_b ? Np : K; b_rows = K; }
        }
    }
    void* const user_C = C;
    if (plan->copy_c && plan->spec.fam != FAM_GENERIC) C = (char*)plan->workspace + plan->c_off;
    auto finish = [&]() -> hgemm_status_t {
        if (hipGetLastError() != hipSuccess) return HGEMM_ERR_LAUNCH;
        if (C == user_C) return HGEMM_OK;
        hipLaunchKernelGGL(copy_back_kernel, dim3((unsigned)((N + 2047) / 2048), (unsigned)std::min<int64_t>(M, 32768)), dim3(256), 0, stream,
                           (const _Float16*)C, plan->lay.ldc, (_Float16*)user_C, plan->ulay.ldc, M, N);
        return hipGetLastError() == hipSuccess ? HGEMM_OK : HGEMM_ERR_LAUNCH;
    };

    // A and B are read in 16-byte chunks; C may start anywhere
    const bool aligned = plan->spec.di || ((((uintptr_t)A) | (plan->any_b ? (uintptr_t)0 : (uintptr_t)B)) & 15) == 0;
    if (plan->spec.fam == FAM_GENERIC || !aligned) {
        const int col_b = row_b ? 0 : 1;
        const int64_t k = plan->uK;                       // of a padded problem too: a copy of A is longer, B need not be
        if (N > (int64_t)64 * 0x7fffffff || (M + 3) / 4 > 65535) {
            // grid.y limit: fold rows into several launches
            for (int64_t mb = 0; mb < M; mb += 4 * 65535) {
                const int64_t rows = std::min<int64_t>(M - mb, 4 * 65535);
                hipLaunchKernelGGL(generic_gemm_kernel, dim3((unsigned)((N + 63) / 64), (unsigned)((rows + 3) / 4)), dim3(256), 0,
                                   stream, (const _Float16*)A + mb * lda, (const _Float16*)B, (_Float16*)C + mb * plan->lay.ldc, rows, N, k,
                                   lda, ldb, plan->lay.ldc, col_b);
            }
        } else {
            hipLaunchKernelGGL(generic_gemm_kernel, dim3((unsigned)((N + 63) / 64), (unsigned)((M + 3) / 4)), dim3(256), 0, stream,
                               (const _Float16*)A, (const _Float16*)B, (_Float16*)C, M, N, k, lda, ldb, plan->lay.ldc, col_b);
        }
        return finish();
    }

    GemmArgs a = plan->args;
    a.A = (const _Float16*)A;
    a.B = (const _Float16*)B;
    a.C = (_Float16*)C;
    a.lda = (int)lda;
    if (!plan->spec.tb) a.ldb = (int)ldb;
    a.b_rows = (int)b_rows;
    a.c_wide = N % 8 == 0 && plan->lay.ldc % 8 == 0 && ((uintptr_t)C & 15) == 0;
    if (plan->skinny) {
        hipLaunchKernelGGL(plan->skinny, skinny_grid(a), dim3(64u * (unsigned)plan->spec.wv), (unsigned)plan->skinny_lds, stream, a);
        if (a.splits > 1 && !plan->spec.fr) {
            if (hipGetLastError() != hipSuccess) return HGEMM_ERR_LAUNCH;
            const int64_t quads = M * ((N + 3) / 4);
            const int blocks = (int)std::min<int64_t>((quads + 255) / 256, 2048);
            hipLaunchKernelGGL(splitk_reduce_kernel, dim3(blocks), dim3(256), 0, stream,
                               (const float*)((const char*)plan->workspace + plan->partial_offset), (_Float16*)C, (int)M, (int)N,
                               part_ld((int)N), (int)plan->lay.ldc, a.c_wide, a.splits);
        }
        return finish();
    }
    const MfmaEntry* e = plan->entry;
    const unsigned wgs = (unsigned)(a.tiles_m * a.tiles_n);
    if (plan->spec.tb) {
        // B (K x N, row-major) -> workspace (N x K, row-major), then the K-contiguous kernel
        hipLaunchKernelGGL(transpose_kernel, dim3((unsigned)((N + 63) / 64), (unsigned)((K + 63) / 64)), dim3(256), 0, stream,
                           (const _Float16*)B, (_Float16*)((char*)plan->workspace + plan->bt_off), (int)K, (int)N, (int)plan->lay.ldb);
        if (hipGetLastError() != hipSuccess) return HGEMM_ERR_LAUNCH;
        a.B = (const _Float16*)((char*)plan->workspace + plan->bt_off);
    }
    const unsigned grid = plan->spec.sm ? (unsigned)(a.dp_tiles + a.sk_workers) : plan->spec.ps ? (unsigned)std::min<int64_t>(wgs, cu_count()) : wgs;
    hipLaunchKernelGGL(a.c_wide && (plan->tn_kernel || a.b_rows == K) ? plan->kernel : plan->kernel_any, dim3(grid, (unsigned)a.splits), dim3(e->threads), plan->kernel_lds, stream, a);
    if (plan->spec.sm) {
        if (hipGetLastError() != hipSuccess) return HGEMM_ERR_LAUNCH;
        hipLaunchKernelGGL(e->fixup, dim3(wgs - (unsigned)a.dp_tiles, (unsigned)((e->bm * e->bn / 4 + 1023) / 1024)), dim3(256), 0,
                           stream, a);
    } else if (a.splits > 1 && !plan->spec.fr) {
        if (hipGetLastError() != hipSuccess) return HGEMM_ERR_LAUNCH;
        const int64_t quads = M * ((N + 3) / 4);
        const int blocks = (int)std::min<int64_t>((quads + 255) / 256, 2048);
        hipLaunchKernelGGL(splitk_reduce_kernel, dim3(blocks), dim3(256), 0, stream,
                           (const float*)((const char*)plan->workspace + plan->partial_offset), (_Float16*)C, (int)M, (int)N,
                           part_ld((int)N), (int)plan->lay.ldc, a.c_wide, a.splits);
    }
    return finish();
}

hgemm_status_t hgemm_run(hgemm_plan_t plan, const void* A, const void* B, void* C, void* hip_stream)
{
    if (!plan) return HGEMM_ERR_INVALID_ARG;
    return run_plan(plan, A, B, C, hip_stream);
}

// The kernel that runs up to `calls` calls of a plan in one launch (null: each call is a launch of its own).  A launch costs a
// call 2.4 us whatever it computes, and one small problem fills a fraction of the chip.
//   * Only kernels that form and add the products in the plan's own order -- unsplit, 32 x 32 x 16 instructions, k ascending,
//     whatever the tile -- so that every result has the bits that hgemm_run gives it; not those of a specialisation that the
//     caller chose, which is to run as it was asked for.
//   * Operands and result of a call up to 8 MiB: 8 x 256^3 27.7 -> 4.4 us, 16 x 512 x 512 x 1024 106 -> 12, 8 x 1024^3 48 -> 20;
//     above, a call takes 12 us and more and the launch little of it (4 x 1536^3 49.9 -> 43).
//   * Tiles of 128 x 128 where the calls of the launch give every compute unit one (8 x 1024 x 1024 x 256: 8.6 us, in 64 x 64 tiles 11.1;
//     8 x 768^3 12.1 against 13.9), else 64 x 64 (4 x 512 x 512 x 1024, 64 tiles of 128: 5.5 us against 8.8).
static const MfmaEntry* merged_entry(const hgemm_plan_s* p, int64_t calls)
{
    const Spec& s = p->spec;
    if (!p->planned || p->blocked || p->padded || !p->entry || !joins_launches(s, p->M, p->N, p->K)) return nullptr;
    static const MfmaEntry* const large = batch_entry(128);
    static const MfmaEntry* const small = batch_entry(64);
    const int64_t tiles128 = ((p->M + 127) / 128) * ((p->N + 127) / 128);
    return calls * tiles128 >= cu_count() ? large : small;
}

// A call's operands as address ranges: calls that share a launch must not write what another of them reads or writes.
struct CallRanges {
    uintptr_t a0, a1, b0, b1, c0, c1;
};
static bool independent(const CallRanges& x, const CallRanges& y)
{
    auto apart = [](uintptr_t p0, uintptr_t p1, uintptr_t q0, uintptr_t q1) { return p1 <= q0 || q1 <= p0; };
    return apart(x.c0, x.c1, y.c0, y.c1) && apart(x.c0, x.c1, y.a0, y.a1) && apart(x.c0, x.c1, y.b0, y.b1) && apart(y.c0, y.c1, x.a0, x.a1) &&
           apart(y.c0, y.c1, x.b0, x.b1);
}

hgemm_status_t hgemm_run_many(hgemm_plan_t plan, int64_t count, int64_t sets, int64_t first, const void* const* A,
                              const void* const* B, void* const* C, void* hip_stream)
{
    if (!plan || count < 0 || sets < 1 || first < 0 || first >= sets || !A || !B || !C) return HGEMM_ERR_INVALID_ARG;
    if (count <= 1 || sets <= 1 || !merged_entry(plan, 2)) {
        int64_t set = first;
        for (int64_t i = 0; i < count; ++i) {
            const hgemm_status_t st = run_plan(plan, A[set], B[set], C[set], hip_stream);
            if (st != HGEMM_OK) return st;
            if (++set == sets) set = 0;
        }
        return HGEMM_OK;
    }
    BatchArgs g;
    static_cast<GemmArgs&>(g) = plan->args;
    const hgemm_layouts_t& l = plan->lay;
    const size_t a_bytes = ((size_t)(plan->M - 1) * l.lda + plan->K) * 2, c_bytes = ((size_t)(plan->M - 1) * l.ldc + plan->N) * 2;
    const size_t b_bytes = l.b == HGEMM_ROW_MAJOR ? ((size_t)(plan->K - 1) * l.ldb + plan->N) * 2 : ((size_t)(plan->N - 1) * l.ldb + plan->K) * 2;
    CallRanges group[kBatchSets];
    int n = 0;
    auto flush = [&]() -> hgemm_status_t {
        if (n == 0) return HGEMM_OK;
        hgemm_status_t st = HGEMM_OK;
        if (n == 1) {
            st = run_plan(plan, g.set[0].A, g.set[0].B, g.set[0].C, hip_stream);
        } else {
            const MfmaEntry* e = merged_entry(plan, n);
            g.tiles_m = (g.M + e->bm - 1) / e->bm;
            g.tiles_n = (g.N + e->bn - 1) / e->bn;
            g.swizzle = g.tiles_m * g.tiles_n <= 16 ? 0 : plan->spec.gm;
            set_tile_map(g);
            hipLaunchKernelGGL(plan->tn_kernel ? e->batch_tn : e->batch, dim3((unsigned)n, (unsigned)(g.tiles_m * g.tiles_n)), dim3(e->threads), e->lds_bytes,
                               (hipStream_t)hip_stream, g);
            if (hipGetLastError() != hipSuccess) st = HGEMM_ERR_LAUNCH;
        }
        n = 0;
        return st;
    };
    int64_t set = first;
    for (int64_t i = 0; i < count; ++i) {
        const uintptr_t a = (uintptr_t)A[set], b = (uintptr_t)B[set], c = (uintptr_t)C[set];
        const bool wide = a && b && c && ((a | b | c) & 15) == 0 && plan->N % 8 == 0 && l.ldc % 8 == 0;
        const CallRanges r{a, a + a_bytes, b, b + b_bytes, c, c + c_bytes};
        bool joins = wide && n < kBatchSets;
        for (int j = 0; joins && j < n; ++j) joins = independent(r, group[j]);
        if (!joins) {
            const hgemm_status_t st = flush();
            if (st != HGEMM_OK) return st;
        }
        if (wide) {
            group[n] = r;               // one more call of the next launch
            g.set[n] = {(const _Float16*)A[set], (const _Float16*)B[set], (_Float16*)C[set]};
            ++n;
        } else {
            const hgemm_status_t st = run_plan(plan, A[set], B[set], C[set], hip_stream);
            if (st != HGEMM_OK) return st;
        }
        if (++set == sets) set = 0;
    }
    return flush();
}

hgemm_status_t hgemm_run_static(int64_t M, int64_t N, int64_t K, const hgemm_layouts_t* layouts, const void* A, const void* B,
                                void* C, void* hip_stream)
{
    hgemm_plan_s plan;                       // lives on this call's stack; its workspace is the static scratch
    const hgemm_status_t st = init_plan(&plan, M, N, K, layouts, nullptr, true);
    if (st != HGEMM_OK) return st;
    return run_plan(&plan, A, B, C, hip_stream);
}

hgemm_status_t hgemm_destroy(hgemm_plan_t plan)
{
    if (!plan) return HGEMM_OK;
    destroy_blocks(plan);
    if (plan->workspace && !plan->static_ws) {
        if (hipFree(plan->workspace) != hipSuccess) (void)hipGetLastError();
    }
    delete plan;
    return HGEMM_OK;
}

const char* hgemm_status_string(hgemm_status_t status)
{
    switch (status) {
        case HGEMM_OK: return "ok";
        case HGEMM_ERR_INVALID_ARG: return "invalid argument";
        case HGEMM_ERR_UNSUPPORTED: return "unsupported layout, alignment or specialisation";
        case HGEMM_ERR_ALLOC: return "allocation failed";
        case HGEMM_ERR_LAUNCH: return "kernel launch failed";
        case HGEMM_ERR_ARCH: return "device is not gfx950";
        case HGEMM_ERR_WORKSPACE: return "problem needs more scratch than the static buffer holds";
    }
    return "unknown status";
}

hgemm_status_t hgemm_plan_describe(hgemm_plan_t plan, char* buf, size_t n)
{
    if (!plan || !buf || n == 0) return HGEMM_ERR_INVALID_ARG;
    std::string s;
    if (plan->blocked) {
        char head[96];
        snprintf(head, sizeof head, "blocks,rows=%lld,cols=%lld%s: ", (long long)plan->block_m, (long long)plan->block_n, plan->blocked_bt ? ",bt=1" : "");
        const hgemm_plan_s* q = plan->sub[0][0] ? plan->sub[0][0] : plan->sub[1][0] ? plan->sub[1][0] : plan->sub[0][1] ? plan->sub[0][1] : plan->sub[1][1];
        s = std::string(head) + (q ? spec_to_string(q->spec) : std::string("?"));
    } else {
        s = spec_to_string(plan->spec) + (plan->padded || (plan->spec.di && plan->planned) ? ",pad=1" : "");
    }
    if (s.size() + 1 > n) { buf[0] = '\0'; return HGEMM_ERR_INVALID_ARG; }
    memcpy(buf, s.c_str(), s.size() + 1);
    return HGEMM_OK;
}

size_t hgemm_plan_workspace_bytes(hgemm_plan_t plan)
{
    if (!plan) return 0;
    size_t bytes = plan->workspace_bytes;
    for (const auto& row : plan->sub)
        for (const hgemm_plan_s* q : row)
            if (q) bytes += q->workspace_bytes;
    return bytes;
}

hgemm_status_t hgemm_plan_launch_info(hgemm_plan_t plan, int64_t* workgroups, int64_t* lds_bytes, int64_t* threads)
{
    if (!plan) return HGEMM_ERR_INVALID_ARG;
    if (plan->blocked) {                     // the figures of the most frequent kind of block
        for (const auto& row : plan->sub)
            for (hgemm_plan_s* q : row)
                if (q) return hgemm_plan_launch_info(q, workgroups, lds_bytes, threads);
        return HGEMM_ERR_INVALID_ARG;
    }
    int64_t wg, lds, th;
    if (plan->skinny) {
        const dim3 grid = skinny_grid(plan->args);
        wg = (int64_t)grid.x * grid.y;
        lds = plan->spec.ra ? 2 * kStripWaves * (plan->M <= 16 ? 1 : 2) * 1024 : plan->skinny_lds ? plan->skinny_lds : 4 * 16 * (kSkinnyCols + 4) * 4;
        th = 64 * plan->spec.wv;
    } else if (plan->entry) {
        wg = plan->spec.sm ? (int64_t)plan->args.dp_tiles + plan->args.sk_workers
                           : (int64_t)plan->args.tiles_m * plan->args.tiles_n * plan->args.splits;
        if (plan->spec.ps) wg = std::min<int64_t>(wg, cu_count());
        lds = plan->kernel_lds;
        th = plan->entry->threads;
    } else {
        wg = ((plan->N + 63) / 64) * ((plan->M + 3) / 4);
        lds = 0;
        th = 256;
    }
    if (workgroups) *workgroups = wg;
    if (lds_bytes) *lds_bytes = lds;
    if (threads) *threads = th;
    return HGEMM_OK;
}

const char* hgemm_spec_help(void)
{
    // built once, inside the initialiser of a function-local static (thread-safe since C++11)
    static const std::string text = [] {
        std::string t =
            "generic\n"
            "    one thread per element, any shape, alignment and layout\n"
            "skinny,sk=SPLITS[,fr=1][,wv=WAVES][,nr=ROWS][,mr=ROWS][,ra=1]\n"
            "    memory-bound kernel for M <= 64 rows of A (row-major B): workgroups of wv = 4 (default), 8 or 16 waves\n"
            "    take 128 columns and a K slab each and stream it in steps of 16 * wv rows; a wave takes 16 rows of a\n"
            "    step, transposes its 4 x 8 blocks in registers for 16x16x16 matrix-core instructions (M on a 16-wide\n"
            "    side; no LDS and no barrier in the main loop), the waves' sums meet once at the end; slabs are summed in\n"
            "    slab order by the split-K reduction launch or, with fr = 1, by the workgroup that arrives last.\n"
            "    Column-major B (K contiguous): a workgroup takes nr = 16, 32, 48 or 64 rows of B (columns of C; default: one strip for\n"
            "    every compute unit up to 12288 columns, narrower where these waves and rows of A have no such kernel), its waves take chunks\n"
            "    of 64 k of them in turn, copied to LDS of their own; sk splits K further across workgroups.  mr = 16, 32, 48 or 64 (with\n"
            "    sk = 1, any M; above 32 four or eight waves): a workgroup takes mr rows of A only.  A row-major B has such strips of\n"
            "    32 columns too: nr=32 with mr = 16 or 32, four waves.  ra = 1 (with sk = 1, wv = 8; M <= 32, K <= 8192, above 16 rows 4096): A stays\n"
            "    in registers, one workgroup per compute unit walks strips of 16 rows of B\n"
            "mfma,bm=BM,bn=BN,bk=BK,wm=WM,wn=WN,st=STAGES[,pf=PREFETCH][,sk=SPLITS][,gm=GROUP][,tb=1][,sm=1][,fr=1][,ps=1][,ac=16][,mi=16][,ph=1][,di=1]\n"
            "    pipelined 32x32x16 MFMA kernel; BMxBN tile per workgroup, WMxWN wavefronts, STAGES LDS buffers,\n"
            "    pf = register prefetch distance in k-steps (1 = ping-pong, 3 = four fragment sets),\n"
            "    sk = split-K factor (fp32 partials + ordered reduction), gm = tile-order group height (0 = row-major),\n"
            "    tb = 1: copy row-major B transposed into the workspace first and run the K-contiguous kernel,\n"
            "    fr = 1: with sk > 1, the reduction is fused into the kernel: every workgroup stores its fp32 plane, the one\n"
            "            that arrives last at a tile sums the planes in split order (same bits as the two-launch form)\n"
            "    ps = 1: persistent: one workgroup per compute unit walks tiles wg, wg + grid, ...; the copies of the next\n"
            "            tile's first K-tiles start under the last K-tiles of the current one\n"
            "    sm = 1: stream-K (whole waves of tiles one per workgroup, the remaining tiles' K iterations dealt\n"
            "            evenly to one more workgroup per CU, fp32 partial tiles summed in k order by a second kernel)\n"
            "    ac = 16: 16-bit accumulator: the running sums are rounded to fp16 after every matrix-core instruction\n"
            "            (16 products); explicit specs only, with sk = 1 and without sm, ps, fr; never chosen by hgemm_plan,\n"
            "            which always accumulates in fp32 over all of K\n"
            "    di = 1: operands at any element's address, with any N and K of at least 8: loaded through registers, zeros behind K\n"
            "            put in on the way (two stages, 32x32x16 instructions); sk and fr allowed, no sm, ps, ph, ac, tb\n"
            "    pad = 1 in a description: N, K or a leading dimension is not a multiple of 8 and the kernel runs on\n"
            "            zero-padded packed copies, held in the plan's workspace, of those of A and B whose rows are not whole\n"
            "            aligned 16-byte chunks, or, with di = 1, pads them on their way through registers (decided by hgemm_plan from the shape)\n"
            "    compiled (bm,bn,bk,wm,wn,st,pf):";
        for (const MfmaEntry& e : registry()) {
            if (e.deep || e.mi != 32) continue;
            char b[64];
            snprintf(b, sizeof b, " (%d,%d,%d,%d,%d,%d,%d)", e.bm, e.bn, e.bk, e.wm, e.wn, e.st, e.pf);
            t += b;
        }
        t += "\n"
             "    deep-staged, pf longer than a K-tile (bk = 32, pf = 3: fragment reads run up to two K-tiles ahead, st stages of\n"
             "    32 k each keep st - 1 K-tiles of copies in flight); one full-K tile per workgroup only: sk = 1, no sm, ps, fr, ac\n"
             "    deep (bm,bn,bk,wm,wn,st,pf):";
        for (const MfmaEntry& e : registry()) {
            if (!e.deep || e.mi != 32) continue;
            char b[64];
            snprintf(b, sizeof b, " (%d,%d,%d,%d,%d,%d,%d)", e.bm, e.bn, e.bk, e.wm, e.wn, e.st, e.pf);
            t += b;
        }
        t += "\n"
             "    mi = 16: v_mfma_f32_16x16x32_f16 instead of v_mfma_f32_32x32x16_f16 (a k-step is then 32 k); one full-K tile per\n"
             "    workgroup only, like the deep-staged ones\n"
             "    mi16 (bm,bn,bk,wm,wn,st,pf):";
        for (const MfmaEntry& e : registry()) {
            if (e.mi != 16) continue;
            char b[64];
            snprintf(b, sizeof b, " (%d,%d,%d,%d,%d,%d,%d)", e.bm, e.bn, e.bk, e.wm, e.wn, e.st, e.pf);
            t += b;
        }
        t += "\n"
             "    ph = 1: the phased schedule of the same tile and waves: a K-tile of 64 is multiplied in four phases, one quadrant of C\n"
             "    each, every phase reads one half tile and refills another (two stages, 16x16x32 instructions); sk allowed, no sm,\n"
             "    ps, fr, ac, tb\n"
             "    phased (bm,bn,bk,wm,wn,st,pf,mi):";
        for (const MfmaEntry& e : registry()) {
            if (!e.phased) continue;
            char b[64];
            snprintf(b, sizeof b, " (%d,%d,%d,%d,%d,%d,%d,%d)", e.bm, e.bn, e.bk, e.wm, e.wn, e.st, e.pf, e.mi);
            t += b;
        }
        t += "\n    direct (bm,bn,bk,wm,wn,st,pf):";
        for (const MfmaEntry& e : registry()) {
            if (!e.direct) continue;
            char b[64];
            snprintf(b, sizeof b, " (%d,%d,%d,%d,%d,%d,%d)", e.bm, e.bn, e.bk, e.wm, e.wn, e.st, e.pf);
            t += b;
        }
        t += "\n";
        return t;
    }();
    return text.c_str();
}

hgemm_status_t hgemm_candidates(int64_t M, int64_t N, int64_t K, const hgemm_layouts_t* layouts, char* buf, size_t n)
{
    if (!buf || n == 0 || M < 0 || N < 0 || K < 0) return HGEMM_ERR_INVALID_ARG;
    hgemm_layouts_t l;
    if (layouts) l = *layouts; else { l.a = l.b = l.c = HGEMM_ROW_MAJOR; l.lda = l.ldb = l.ldc = 0; }
    if (l.lda == 0) l.lda = K;
    if (l.ldb == 0) l.ldb = (l.b == HGEMM_ROW_MAJOR) ? N : K;
    if (l.ldc == 0) l.ldc = N;
    std::string out;
    if (!fast_path_ok(M, N, K, l) || M == 0 || N == 0 || K == 0) {
        out = "generic\n";
    } else {
        const int64_t CUS = cu_count();
        if (l.b == HGEMM_ROW_MAJOR && M <= kSkinnyMaxM) {       // few rows: the streaming family competes
            for (int eff : skinny_split_candidates(N, K)) {
                for (int fr = 0; fr <= ((eff > 1 && fused_delta_us(M, N, eff) < 1.0) ? 1 : 0); ++fr) {
                    for (int wv : {4, 8, 16}) {
                        if (wv == 16 && M > 32) continue;
                        Spec s;
                        s.fam = FAM_SKINNY; s.sk = (int)eff; s.fr = fr; s.wv = wv;
                        if (effective_splits((K + skinny_step(s) - 1) / skinny_step(s), eff) != eff) continue;
                        out += spec_to_string(s);
                        out += "\n";
                    }
                }
            }
        }
        if (l.b == HGEMM_COL_MAJOR && M <= kSkinnyMaxM) {       // the streaming family for K-contiguous B: N / 16 workgroups before any split
            for (int nr : {16, 32, 48, 64})      // 16 as the default where that is what it is
                for (int wv : {4, 8, 16}) {
                    if (!skinny_tn_exists(wv, row_blocks_of_a(M), nr / 16, false)) continue;
                    if (nr > 16 && (N + nr - 1) / nr < CUS / 2) continue;             // too few workgroups to be worth timing
                    int64_t last = 0;
                    for (int sk : {1, 2, 4, 8, 16}) {
                        Spec s;
                        s.fam = FAM_SKINNY; s.wv = wv; s.nr = nr;
                        if (nr == 16) { s.nr = 0; if (sk == 1 && strip_rows(s, M, N) != 16) s.nr = 16; }
                        const int64_t eff = effective_splits((K + skinny_step(s, true) - 1) / skinny_step(s, true), sk);
                        if (eff == last || ((N + nr - 1) / nr) * eff > 64 * CUS) continue;
                        last = eff;
                        for (int fr = 0; fr <= (eff > 1 ? 1 : 0); ++fr) {
                            s.sk = (int)eff; s.fr = fr;
                            out += spec_to_string(s);
                            out += "\n";
                        }
                    }
                }
        }
        if (l.b == HGEMM_COL_MAJOR && M > 16 && M <= 512)       // blocks of rows of A: one workgroup for most compute units
            for (int mr : {16, 32, 48, 64})
                for (int nr : {16, 32, 48, 64}) {
                    const int64_t wgs = ((M + mr - 1) / mr) * ((N + nr - 1) / nr);
                    if (mr >= M + 16 || wgs > CUS || wgs < CUS / 2) continue;
                    Spec s;
                    s.fam = FAM_SKINNY; s.mr = mr; s.nr = nr;
                    out += spec_to_string(s);
                    out += "\n";
                }
        if (l.b == HGEMM_COL_MAJOR && M <= 32 && N >= 16 * CUS && skinny_strips(M <= 16 ? 1 : 2, K)) out += "skinny,sk=1,wv=8,ra=1\n";
        for (const MfmaEntry& e : registry()) {
            if (!tile_fits_problem(e, M, N)) continue;
            const int64_t t = ((M + e.bm - 1) / e.bm) * ((N + e.bn - 1) / e.bn);
            const int64_t ktiles = (K + e.bk - 1) / e.bk;
            if (e.deep) {                                       // one full-K tile per workgroup; worth timing once the chip is full
                if (t < CUS / 2 || ktiles < 2 * e.st) continue;
                for (int gm : {8, 0, 4, 16}) {
                    if (gm != 8 && (t < 2 * CUS)) continue;
                    Spec s;
                    s.fam = FAM_MFMA; s.bm = e.bm; s.bn = e.bn; s.bk = e.bk; s.wm = e.wm; s.wn = e.wn; s.st = e.st; s.pf = e.pf; s.mi = e.mi; s.sk = 1; s.gm = gm;
                    out += spec_to_string(s);
                    out += "\n";
                }
                continue;
            }
            const SplitFactors sks = split_candidates(t, ktiles);
            if (t % CUS != 0 && ktiles >= 4 && e.bm >= 64 && e.bn >= 64) {
                Spec s;
                s.fam = FAM_MFMA; s.bm = e.bm; s.bn = e.bn; s.bk = e.bk; s.wm = e.wm; s.wn = e.wn; s.st = e.st; s.pf = e.pf; s.mi = e.mi; s.sk = 1; s.gm = 8; s.sm = 1;
                out += spec_to_string(s);
                out += "\n";
            }
            for (int sk : sks) {
                for (int gm : {8, 0, 4, 16}) {
                    if (gm != 8 && (t < 2 * CUS)) continue;      // order matters only when tiles outnumber CUs
                    Spec s;
                    s.fam = FAM_MFMA; s.bm = e.bm; s.bn = e.bn; s.bk = e.bk; s.wm = e.wm; s.wn = e.wn; s.st = e.st; s.pf = e.pf; s.mi = e.mi; s.sk = sk; s.gm = gm;
                    out += spec_to_string(s);
                    out += "\n";
                    if (sk == 1 && gm == 8 && e.persist && t > CUS && ktiles >= e.st) {      // the same tiles walked by persistent workgroups
                        s.ps = 1;
                        out += spec_to_string(s);
                        out += "\n";
                        s.ps = 0;
                    }
                    if (e.phased) {                              // the same tiles on the phased schedule
                        s.ph = 1;
                        out += spec_to_string(s);
                        out += "\n";
                        s.ph = 0;
                    }
                    if (sk > 1 && gm == 8 && fused_delta_us(M, N, sk) < 1.0) {   // the same split with the reduction fused into the kernel
                        s.fr = 1;
                        out += spec_to_string(s);
                        out += "\n";
                        s.fr = 0;
                    }
                    // row-major B, tall problem: paying one transposing copy of B can be cheaper than
                    // transposing reads in every workgroup
                    if (l.b == HGEMM_ROW_MAJOR && gm == 8 && M >= 1024 && e.bm >= 128 && e.bn >= 128) {
                        s.tb = 1;
                        out += spec_to_string(s);
                        out += "\n";
                    }
                }
            }
        }
    }
    if (out.size() + 1 > n) { buf[0] = '\0'; return HGEMM_ERR_INVALID_ARG; }
    memcpy(buf, out.c_str(), out.size() + 1);
    return HGEMM_OK;
}

hgemm_status_t hgemm_predict_us(int64_t M, int64_t N, int64_t K, const char* spec, double* us)
{
    if (!spec || !us || M <= 0 || N <= 0 || K <= 0) return HGEMM_ERR_INVALID_ARG;
    Spec s;
    if (!parse_spec(spec, &s)) return HGEMM_ERR_INVALID_ARG;
    return predict_spec_us(M, N, K, s, us) ? HGEMM_OK : HGEMM_ERR_UNSUPPORTED;
}

int64_t hgemm_tiles(int64_t dim, int64_t tile) { return (dim < 0 || tile <= 0) ? -1 : (dim + tile - 1) / tile; }
int64_t hgemm_padded(int64_t dim, int64_t tile) { return (dim < 0 || tile <= 0) ? -1 : ((dim + tile - 1) / tile) * tile; }

int64_t hgemm_tile_of_workgroup(int64_t wg, int64_t tiles_m, int64_t tiles_n, int64_t swizzle)
{
    if (tiles_m <= 0 || tiles_n <= 0 || wg < 0 || wg >= tiles_m * tiles_n || swizzle < 0) return -1;
    const int64_t tile = tile_of_workgroup(wg, tiles_m, tiles_n, swizzle);
    // the kernels use the multiplication form of the same map: report a disagreement instead of hiding it
    if (tiles_m * tiles_n < ((int64_t)1 << 24)) {
        GemmArgs a{};
        a.tiles_m = (int)tiles_m;
        a.tiles_n = (int)tiles_n;
        a.swizzle = (int)std::min<int64_t>(swizzle, tiles_m);
        set_tile_map(a);
        unsigned tm = 0, tn = 0;
        tile_coords((unsigned)wg, a, tm, tn);
        if ((int64_t)tm * tiles_n + tn != tile) return -2;
    }
    return tile;
}

hgemm_status_t hgemm_calibrate_mfma(int64_t iters, void* hip_stream, double* ms, double* flop)
{
    if (!ms || !flop || iters <= 0 || iters > (1 << 24)) return HGEMM_ERR_INVALID_ARG;
    hipStream_t stream = (hipStream_t)hip_stream;
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) { (void)hipGetLastError(); return HGEMM_ERR_ARCH; }
    float* out = nullptr;
    if (hipMalloc(&out, 4) != hipSuccess) { (void)hipGetLastError(); return HGEMM_ERR_ALLOC; }
    hipEvent_t e0, e1;
    hipEventCreate(&e0);
    hipEventCreate(&e1);
    const int blocks = prop.multiProcessorCount * 2;
    hipLaunchKernelGGL(calib_mfma_kernel, dim3(blocks), dim3(256), 0, stream, out, (int)iters);   // warm-up
    hipEventRecord(e0, stream);
    hipLaunchKernelGGL(calib_mfma_kernel, dim3(blocks), dim3(256), 0, stream, out, (int)iters);
    hipEventRecord(e1, stream);
    hipError_t err = hipEventSynchronize(e1);
    float t = 0.f;
    if (err == hipSuccess) err = hipEventElapsedTime(&t, e0, e1);
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    hipFree(out);
    if (err != hipSuccess) { (void)hipGetLastError(); return HGEMM_ERR_LAUNCH; }
    *ms = t;
    *flop = (double)blocks * 4.0 * (double)iters * 4.0 * 32768.0;    // 4 waves x 4 MFMAs of 32*32*16*2 flop
    return HGEMM_OK;
}

hgemm_status_t hgemm_calibrate_hbm_read(const void* src, size_t bytes, void* hip_stream, double* ms)
{
    if (!src || !ms || bytes < 16 || (((uintptr_t)src) & 15)) return HGEMM_ERR_INVALID_ARG;
    hipStream_t stream = (hipStream_t)hip_stream;
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) { (void)hipGetLastError(); return HGEMM_ERR_ARCH; }
    uint32_t* out = nullptr;
    if (hipMalloc(&out, 4) != hipSuccess) { (void)hipGetLastError(); return HGEMM_ERR_ALLOC; }
    hipEvent_t e0, e1;
    hipEventCreate(&e0);
    hipEventCreate(&e1);
    const int blocks = prop.multiProcessorCount * 8;
    hipEventRecord(e0, stream);
    hipLaunchKernelGGL(calib_read_kernel, dim3(blocks), dim3(256), 0, stream, (const uint4*)src, bytes / 16, out);
    hipEventRecord(e1, stream);
    hipError_t err = hipEventSynchronize(e1);
    float t = 0.f;
    if (err == hipSuccess) err = hipEventElapsedTime(&t, e0, e1);
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    hipFree(out);
    if (err != hipSuccess) { (void)hipGetLastError(); return HGEMM_ERR_LAUNCH; }
    *ms = t;
    return HGEMM_OK;
}

}  // extern "C"
