// C-ABI entry points of the device path: argument checks, launch-shape
// heuristic, dispatch.  Contract: include/kmq.h.
#include <cstdlib>
#include <hip/hip_runtime.h>

#include "kmq.h"
#include "kmq_internal.h"
#include "kmq_launch.h"

namespace kmq {

// On the canonical layout a batch above 1 runs the batch-1 table kernel, where the shape has one, over a
// grid of (row group, group of up to four columns) workgroups in ONE launch: the workgroups that share rows of W sit next to
// each other on one XCD, so W still comes from memory once and the other columns find it in that L2 (the
// tiled layout with its matrix-core kernel remains the fastest route for batch > 1: it also decodes each
// weight once).  Which batches take several columns a workgroup: kmq_lut_columns.hip.  Measured (us), table kernel /
// shape-agnostic: 9216x3072 1-bit, batch 4: 6.4 / 21.7; 14336x4096 2-bit, batch 16: 27.4 / 121; 4096x4096 4-bit,
// batch 4: 6.6 / 12.8.  (Builds with -DKMQ_TUNING read a cap on the batch from KMQ_PER_COLUMN_MAX in the environment,
// for sweeps.)
static bool per_column_faster(int M) {
#ifdef KMQ_TUNING
    static const char* const v = std::getenv("KMQ_PER_COLUMN_MAX");
    static const int cap = v ? std::atoi(v) : KMQ_MAX_BATCH;
#else
    constexpr int cap = KMQ_MAX_BATCH;
#endif
    return M >= 2 && M <= cap;
}

// Where the matrix-core kernel for any row length (kmq_mfma_any.h) takes a product from the vector kernels of the canonical layout.
// It decodes every weight once for the whole batch, so a shape-agnostic per-row product (K no multiple of 32, or a batch on few
// long rows) is always its (3-bit 5001 x 4101, batch 1 / 3 / 16: 41.0 / 111.0 / 567 -> 7.6 / 8.0 / 11.8 us).  The other vector
// kernels spread a product over more workgroups than one per 16 rows: with at most 256 blocks of 16 rows (one a CU) it takes a
// time that K, the batch group and the bit-width set, whatever the number of rows, and theirs grows with N * K * M from
// a floor.  Both are estimated from straight lines through measurements (us, vector / this):
//   K in rounds, batch >= 2: 4-bit 13824 columns, batch 8: 64 rows 4.4 / 11.0, 512 14.4 / 11.9, 2048 28.7 / 12.5; 1-bit 6912
//     columns, batch 4: 512 rows 4.1 / 5.0, 2048 7.7 / 4.9
//   block-scaled, batch 1: 4-bit 3648 columns: 1024 rows 3.8 / 7.1, 4096 7.2 / 7.6; 1-bit 11008 columns: 1024 5.9 / 6.2, 4096
//     13.2 / 6.8
//   block-scaled with a table kernel, batch 8: 4-bit 8192 columns: 256 rows 4.7 / 9.7, 1024 8.0 / 9.9, 4096 20.0 / 10.5
// With more rows it is always faster from batch 2 (K in rounds; 2-bit 4096 x 11008, batch 16: 45.3 -> 12.3), at every batch
// (block-scaled without a table kernel) and from batch 3 on (with one; 143 drawn shapes of 4097 to 8192 rows, 2048 to 14336 columns: 6 % less time at
// the least; 2-bit 4928 x 8192, batch 3: 9.9 -> 8.1).
// The lines were drawn against table kernels of two columns a workgroup, and with this kernel's last tile fetched element by element and its lines of words asked for
// more than once.  Block-scaled with a table kernel, 700 shapes (256..8192 rows, batch 2..16): the slower side by more than 10 % in 43, 1.7 % over the faster one on
// average; all but one of the 43 are table kernels (2-bit 896 x 14336, batch 14: 15.9 taken, 9.5 the other), where a column is its batch-1 result bit for bit.
// By time alone the lines against the rounds would be lower since the words come by whole lines and a last piece as one load (costs of 0.85 per column, 0.4 for a
// last tile: 500 drawn shapes of 64 to 4096 rows whose route that changes, 24 % less time, 7 of them 4 to 16 % more).  They are not, for two reasons: up to them a
// column is its batch-1 result bit for bit, and the 32-bit sums of the rounds are rounded less (rows that cancel, 1500 such shapes, root mean square of this
// kernel over theirs: 2 and 3 bits 1.03, from 40 tiles on 1.01, 4 bits 1.07).
// Table kernels specialised on K keep per-row batches: their columns are the batch-1 results bit for bit.
constexpr int64_t kAnyOneRound = 256 * 16;
struct AnyCost { double start, per_k[3]; };               // us; us per 1000 columns at batches up to 4, 8, 16
static double any_length_us(int64_t K, int bits, int M, bool scaled) {
    static const AnyCost cost[2][4] = {{{3.0, {0.30, 0.45, 0.72}}, {2.8, {0.26, 0.45, 0.75}}, {2.8, {0.45, 0.58, 0.85}}, {3.6, {0.53, 0.68, 0.95}}},
                                       {{2.7, {0.38, 0.45, 0.62}}, {2.9, {0.45, 0.53, 0.68}}, {2.6, {0.65, 0.73, 0.90}}, {4.1, {0.70, 0.77, 0.90}}}};
    static const double tail[3] = {0.8, 1.3, 2.5};        // a last tile that K does not fill
    const int g = M <= 4 ? 0 : M <= 8 ? 1 : 2;
    const AnyCost& c = cost[scaled ? 1 : 0][bits - 1];
    return c.start + c.per_k[g] * 1e-3 * static_cast<double>(K) + (K % 256 ? tail[g] : 0.0);
}
static double from_floor(double floor, double start, double each, double work) {
    const double t = start + each * work;
    return t > floor ? t : floor;
}
static double millions(int64_t N, int64_t K, int M) { return 1e-6 * static_cast<double>(N) * static_cast<double>(K) * M; }
// against the table kernel that walks K in rounds
static bool any_beats_rounds(int64_t N, int64_t K, int bits, int M) {
    static const double each[4] = {0.10, 0.105, 0.12, 0.19};
    const int64_t k = K > 2048 ? K : 2048;                // (shorter rows cost it as much; large matrices get a better launch shape)
    const double work = millions(N, k, M) * (N * K > (int64_t(24) << 20) ? 0.75 : 1.0);
    return M >= 2 && (N > kAnyOneRound || any_length_us(K, bits, M, false) < from_floor(bits == 3 ? 4.3 : 4.0, 2.5, each[bits - 1], work));
}
// against the specialised table kernels, block-scaled
static bool any_beats_scaled_table(int64_t N, int64_t K, int bits, int M) {
    static const double each[4] = {0.045, 0.055, 0.07, 0.105};
    return M >= 3 && (N > kAnyOneRound || any_length_us(K, bits, M, true) < from_floor(3.7, 2.0, each[bits - 1], millions(N, K, M)));
}
// against a wave per row and a lane per block (from batch 4 on its columns' latencies alone are longer, and from batch 2 on where
// they do not fit the first-level cache: 4-bit 1088 x 7808, batch 3: 14.2 against 10.4)
static bool any_beats_block_generic(int64_t N, int64_t K, int bits, int M) {
    if (bits > 4) return false;
    if (M >= 4 || N > kAnyOneRound || (M >= 2 && K > 4096)) return true;
    const double rounds = static_cast<double>((K / KMQ_BLOCK + 63) / 64);
    const double latency = 2.6 + (M == 1 ? 0.9 : 2.6 + 0.9 * (M - 2)) * rounds;
    return any_length_us(K, bits, M, true) < from_floor(latency, 1.9, 0.28 * (1 + 0.7 * (M - 1)), millions(N, K, 1));
}
static Plan any_length_plan(int bits, bool scaled) {
    static const char* const names[2][4] = {{"mfma_any_b1", "mfma_any_b2", "mfma_any_b3", "mfma_any_b4"},
                                            {"mfma_any_sc_b1", "mfma_any_sc_b2", "mfma_any_sc_b3", "mfma_any_sc_b4"}};
    return Plan{kVariantMfmaAny, -1, 0, names[scaled ? 1 : 0][bits - 1]};
}

// Launch-shape heuristic (the paper autotunes chunk shapes per problem, App. E
// "Kernel implementations"; here the choice is a static function of the shape).
Plan make_plan(int64_t N, int64_t K, int bits, int M, int layout, bool scaled) {
    Plan p{kVariantInvalid, -1, 0, "invalid"};
    if (!bits_valid(bits) || !dims_valid(N, K) || M < 1 || M > KMQ_MAX_BATCH) return p;
    if (layout != KMQ_LAYOUT_CANONICAL && layout != KMQ_LAYOUT_TILED && layout != KMQ_LAYOUT_ROWLANE) return p;
    if (layout == KMQ_LAYOUT_ROWLANE) {
        if (scaled || !rowlane_valid(bits, K) || !rowlane_has_kernel(K, bits, M)) return p;
        static const char* const names[2][2] = {{"rowlane_b1", "rowlane_b2"}, {"rowlane_loop_b1", "rowlane_loop_b2"}};
        return Plan{kVariantRowlane, -1, 0, names[rowlane_loops(K, bits) ? 1 : 0][bits - 1]};
    }
    if (scaled) {
        if (K % KMQ_BLOCK != 0) return p;
        if (layout == KMQ_LAYOUT_TILED) {
            // matrix-core kernel; its LDS holds the scales of at most 256 blocks of K per row
            if (!tiled_valid(bits, K) || K > 256 * KMQ_BLOCK) return p;
            static const char* const names[4] = {"mfma_sc_b1", "mfma_sc_b2", "mfma_sc_b3", "mfma_sc_b4"};
            if (!mfma_takes(N, K, bits, M, true)) return any_length_plan(bits, true);
            return Plan{kVariantMfma, -1, 0, names[bits - 1]};
        }
        if (M == 1 || per_column_faster(M)) {
            const int l = lut_find(N, K, bits, layout, true);
            if (l >= 0 && any_beats_scaled_table(N, K, bits, M)) return any_length_plan(bits, true);
            if (l >= 0) return Plan{M == 1 ? kVariantLut : kVariantPerColumn, l, 0, lut_name(l)};
        }
        if (any_beats_block_generic(N, K, bits, M)) return any_length_plan(bits, true);
        return Plan{kVariantBlockGeneric, -1, 0, "blockscaled_generic"};
    }
    if (layout == KMQ_LAYOUT_TILED && !tiled_valid(bits, K)) return p;
    if (layout == KMQ_LAYOUT_TILED) {
        static const char* const names[4] = {"mfma_b1", "mfma_b2", "mfma_b3", "mfma_b4"};
        if (!mfma_takes(N, K, bits, M, false)) return any_length_plan(bits, false);
        if (mfma_kslice_has_kernel(N, K, bits)) return Plan{kVariantMfma, -1, 0, bits == 2 ? "mfma_kslice_b2" : "mfma_kslice_b3"};
        return Plan{kVariantMfma, -1, 0, names[bits - 1]};
    }
    bool use_loop = true, use_table = true;
#ifdef KMQ_TUNING
    static const char* const loop_env = std::getenv("KMQ_LOOP");      // sweeps only: 0 = never, 2 = instead of the specialised kernels
    if (loop_env) { use_loop = loop_env[0] != '0'; use_table = loop_env[0] != '2'; }
#endif
    if (use_table && (M == 1 || per_column_faster(M))) {
        const int l = lut_find(N, K, bits, layout);
        if (l >= 0) return Plan{M == 1 ? kVariantLut : kVariantPerColumn, l, 0, lut_name(l)};
    }
    const int slices = generic_splitk_slices(N, K, layout);
    if (slices > 1)
        return Plan{kVariantGeneric, slices, static_cast<size_t>(slices) * M * N * sizeof(float), "generic_splitk"};
    if (use_loop && (M == 1 || per_column_faster(M)) && lut_loop_has_kernel(N, K, bits, layout) && !any_beats_rounds(N, K, bits, M))
        return Plan{kVariantLutLoop, -1, 0, lut_loop_name(bits)};
    if (bits <= 4) return any_length_plan(bits, false);
    if (mfma_b8_takes(N, K, M)) return Plan{kVariantMfmaB8, -1, 0, "mfma_b8"};
    return Plan{kVariantGeneric, -1, 0, "generic"};
}

// Text of the last HIP error a launch reported on this thread ("" if none).
static thread_local const char* g_last_hip_error = "";

static kmq_status hip_status(hipError_t e) {
    if (e == hipSuccess) return KMQ_OK;
    g_last_hip_error = hipGetErrorString(e);
    return KMQ_ERR_HIP;
}

static bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// library_scratch: the caller brings no workspace; a plan that needs one takes this GPU's share of the
// library's own scratch array (kmq_gemm_smallbatch_noalloc), up to its fixed size.
static kmq_status check_and_run(const GemmArgs& a_in, void* stream, bool library_scratch = false) {
    GemmArgs a = a_in;
    if (!a.W || !a.codebook || !a.X || !a.Y) return KMQ_ERR_NULL;
    if (!bits_valid(a.bits)) return KMQ_ERR_BITS;
    if (!dims_valid(a.N, a.K) || a.M < 1 || a.M > KMQ_MAX_BATCH) return KMQ_ERR_SHAPE;
    if (a.layout != KMQ_LAYOUT_CANONICAL && a.layout != KMQ_LAYOUT_TILED && a.layout != KMQ_LAYOUT_ROWLANE) return KMQ_ERR_LAYOUT;
    if (a.layout == KMQ_LAYOUT_TILED && !tiled_valid(a.bits, a.K)) return KMQ_ERR_LAYOUT;
    if (a.layout == KMQ_LAYOUT_ROWLANE && (!rowlane_valid(a.bits, a.K) || a.scales)) return KMQ_ERR_LAYOUT;
    if (!aligned(a.W, 16) || !aligned(a.X, 16) || !aligned(a.codebook, 4) || !aligned(a.Y, 2)) return KMQ_ERR_ALIGN;
    const bool scaled = a.scales != nullptr;
    if (scaled) {
        if (a.K % KMQ_BLOCK != 0) return KMQ_ERR_SHAPE;
        if (a.layout == KMQ_LAYOUT_TILED && a.K > 256 * KMQ_BLOCK) return KMQ_ERR_LAYOUT;
        if (!aligned(a.scales, 2)) return KMQ_ERR_ALIGN;
    }
    const Plan plan = make_plan(a.N, a.K, a.bits, a.M, a.layout, scaled);
    if (plan.variant == kVariantInvalid) return a.layout == KMQ_LAYOUT_ROWLANE ? KMQ_ERR_LAYOUT : KMQ_ERR_SHAPE;
    if (plan.workspace_bytes > 0 && library_scratch) {
        if (plan.workspace_bytes > KMQ_NOALLOC_SCRATCH_BYTES) return KMQ_ERR_WORKSPACE;
        const hipError_t es = noalloc_scratch(&a.workspace);
        if (es != hipSuccess) return hip_status(es);
        a.workspace_bytes = KMQ_NOALLOC_SCRATCH_BYTES;
    }
    if (plan.workspace_bytes > 0 && (!a.workspace || a.workspace_bytes < plan.workspace_bytes)) return KMQ_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e = hipSuccess;
    switch (plan.variant) {
        case kVariantMfmaAny: {
            static hipError_t (*const launch[4])(const GemmArgs&, hipStream_t) = {launch_canon_b1, launch_canon_b2, launch_canon_b3, launch_canon_b4};
            e = launch[a.bits - 1](a, s);
            break;
        }
        case kVariantMfma: e = launch_mfma(a, s); break;
        case kVariantMfmaB8: e = launch_mfma_b8(a, s); break;
        case kVariantRowlane: e = launch_rowlane(a, s); break;
        case kVariantLut: e = launch_lut_entry(plan.table_index, a, s); break;
        case kVariantPerColumn:                               // one launch, a workgroup per (row group, column)
            e = launch_lut_entry(plan.table_index, a, s);   // K is a multiple of 8 for every table kernel: rows of X stay 16-byte aligned
            break;
        case kVariantLutLoop: e = launch_lut_loop(a, s); break;
        case kVariantBlockGeneric: e = launch_blockscaled_generic(a, s); break;
        default: e = launch_generic(a, s); break;
    }
    return hip_status(e);
}

}  // namespace kmq

extern "C" {

size_t kmq_workspace_bytes(int64_t N, int64_t K, int bits, int M, int layout) {
    return kmq::make_plan(N, K, bits, M, layout).workspace_bytes;
}

const char* kmq_kernel_name(int64_t N, int64_t K, int bits, int M, int layout) {
    return kmq::make_plan(N, K, bits, M, layout).name;
}

kmq_status kmq_gemm_smallbatch(const uint32_t* W, const uint16_t* codebook, const uint16_t* X,
                               uint16_t* Y, int64_t N, int64_t K, int M, int bits, int layout,
                               void* workspace, size_t workspace_bytes, void* hip_stream) {
    const kmq::GemmArgs a{W, codebook, X, Y, N, K, M, bits, layout, workspace, workspace_bytes};
    return kmq::check_and_run(a, hip_stream);
}

kmq_status kmq_gemm_smallbatch_noalloc(const uint32_t* W, const uint16_t* codebook, const uint16_t* X,
                                       uint16_t* Y, int64_t N, int64_t K, int M, int bits, int layout,
                                       void* hip_stream) {
    const kmq::GemmArgs a{W, codebook, X, Y, N, K, M, bits, layout, nullptr, 0};
    return kmq::check_and_run(a, hip_stream, /*library_scratch=*/true);
}

kmq_status kmq_gemv(const uint32_t* W, const uint16_t* codebook, const uint16_t* x, uint16_t* y,
                    int64_t N, int64_t K, int bits, int layout,
                    void* workspace, size_t workspace_bytes, void* hip_stream) {
    const kmq::GemmArgs a{W, codebook, x, y, N, K, 1, bits, layout, workspace, workspace_bytes};
    return kmq::check_and_run(a, hip_stream);
}

kmq_status kmq_gemv_swiglu(const uint32_t* Wgate, const uint16_t* codebook_gate,
                           const uint32_t* Wup, const uint16_t* codebook_up,
                           const uint16_t* x, uint16_t* y, int64_t N, int64_t K, int bits, int layout,
                           void* hip_stream) {
    if (!Wgate || !codebook_gate || !Wup || !codebook_up || !x || !y) return KMQ_ERR_NULL;
    if (!kmq::bits_valid(bits)) return KMQ_ERR_BITS;
    if (!kmq::dims_valid(N, K) || 2 * N > kmq::kMaxDim) return KMQ_ERR_SHAPE;
    const bool rowlane = layout == KMQ_LAYOUT_ROWLANE && kmq::rowlane_pair_has_kernel(K, bits);
    if (layout != KMQ_LAYOUT_CANONICAL && !rowlane) return KMQ_ERR_LAYOUT;
    if (!kmq::aligned(Wgate, 16) || !kmq::aligned(Wup, 16) || !kmq::aligned(x, 16) ||
        !kmq::aligned(codebook_gate, 4) || !kmq::aligned(codebook_up, 4) || !kmq::aligned(y, 2)) return KMQ_ERR_ALIGN;
    kmq::GemmArgs a{Wgate, codebook_gate, x, y, N, K, 1, bits, layout, nullptr, 0};
    a.W2 = Wup;
    a.codebook2 = codebook_up;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (rowlane) return kmq::hip_status(kmq::launch_rowlane_pair(a, s));
    const int l = kmq::lut_find(2 * N, K, bits, layout, false);
    const hipError_t e = l >= 0 ? kmq::launch_lut_entry(l, a, s) : kmq::launch_fused_generic(a, s);
    return kmq::hip_status(e);
}

const char* kmq_kernel_name_swiglu(int64_t N, int64_t K, int bits, int layout) {
    if (!kmq::bits_valid(bits) || !kmq::dims_valid(N, K)) return "invalid";
    if (layout == KMQ_LAYOUT_ROWLANE && kmq::rowlane_pair_has_kernel(K, bits)) return bits == 1 ? "rowlane_pair_b1" : "rowlane_pair_b2";
    if (layout != KMQ_LAYOUT_CANONICAL) return "invalid";
    const int l = kmq::lut_find(2 * N, K, bits, layout, false);
    return l >= 0 ? kmq::lut_name(l) : "pair_generic";
}

kmq_status kmq_gemv_fused(const uint32_t* W, const uint16_t* codebook, const uint16_t* x,
                          int rmsnorm, const uint16_t* norm_weight, float eps, const uint16_t* residual, uint16_t* y,
                          int64_t N, int64_t K, int bits, int layout, void* hip_stream) {
    if (!W || !codebook || !x || !y) return KMQ_ERR_NULL;
    if (!kmq::bits_valid(bits)) return KMQ_ERR_BITS;
    if (!kmq::dims_valid(N, K) || (rmsnorm && !(eps >= 0.f)) || (rmsnorm != 0 && rmsnorm != 1)) return KMQ_ERR_SHAPE;
    if (!rmsnorm) norm_weight = nullptr;
    if (layout != KMQ_LAYOUT_CANONICAL) return KMQ_ERR_LAYOUT;
    if (!kmq::aligned(W, 16) || !kmq::aligned(x, 16) || !kmq::aligned(codebook, 4) || !kmq::aligned(y, 2) ||
        (norm_weight && !kmq::aligned(norm_weight, 16)) || (residual && !kmq::aligned(residual, 2))) return KMQ_ERR_ALIGN;
    kmq::GemmArgs a{W, codebook, x, y, N, K, 1, bits, layout, nullptr, 0};
    a.norm = rmsnorm != 0;
    a.norm_w = norm_weight;
    a.eps = eps;
    a.residual = residual;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int l = kmq::lut_find(N, K, bits, layout, false);
    hipError_t e;
    if (l >= 0 && kmq::lut_has_fusions(l)) e = kmq::launch_lut_entry(l, a, s);
    else if (!rmsnorm && kmq::lut_loop_has_kernel(N, K, bits, layout)) e = kmq::launch_lut_loop(a, s);   // residual behind: the K-loop table kernel
    else e = kmq::launch_fused_generic(a, s);
    return kmq::hip_status(e);
}

kmq_status kmq_gemv_swiglu_rmsnorm(const uint32_t* Wgate, const uint16_t* codebook_gate,
                                   const uint32_t* Wup, const uint16_t* codebook_up,
                                   const uint16_t* x, const uint16_t* norm_weight, float eps, uint16_t* y,
                                   int64_t N, int64_t K, int bits, int layout, void* hip_stream) {
    if (!Wgate || !codebook_gate || !Wup || !codebook_up || !x || !y) return KMQ_ERR_NULL;
    if (!kmq::bits_valid(bits)) return KMQ_ERR_BITS;
    if (!kmq::dims_valid(N, K) || 2 * N > kmq::kMaxDim || !(eps >= 0.f)) return KMQ_ERR_SHAPE;
    if (layout != KMQ_LAYOUT_CANONICAL) return KMQ_ERR_LAYOUT;
    if (!kmq::aligned(Wgate, 16) || !kmq::aligned(Wup, 16) || !kmq::aligned(x, 16) || (norm_weight && !kmq::aligned(norm_weight, 16)) ||
        !kmq::aligned(codebook_gate, 4) || !kmq::aligned(codebook_up, 4) || !kmq::aligned(y, 2)) return KMQ_ERR_ALIGN;
    kmq::GemmArgs a{Wgate, codebook_gate, x, y, N, K, 1, bits, layout, nullptr, 0};
    a.W2 = Wup;
    a.codebook2 = codebook_up;
    a.norm = true;
    a.norm_w = norm_weight;
    a.eps = eps;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int l = kmq::lut_find(2 * N, K, bits, layout, false);
    const hipError_t e = (l >= 0 && kmq::lut_has_fusions(l)) ? kmq::launch_lut_entry(l, a, s) : kmq::launch_fused_generic(a, s);
    return kmq::hip_status(e);
}

const char* kmq_kernel_name_fused(int64_t N, int64_t K, int bits, int layout, int pair) {
    if (!kmq::bits_valid(bits) || !kmq::dims_valid(N, K) || layout != KMQ_LAYOUT_CANONICAL) return "invalid";
    const int l = kmq::lut_find(pair ? 2 * N : N, K, bits, layout, false);
    return (l >= 0 && kmq::lut_has_fusions(l)) ? kmq::lut_name(l) : "fused_generic";
}

kmq_status kmq_gemm_smallbatch_blockscaled(const uint32_t* W, const uint16_t* codebook, const uint16_t* scales,
                                           const uint16_t* X, uint16_t* Y, int64_t N, int64_t K, int M, int bits,
                                           int layout, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!scales) return KMQ_ERR_NULL;
    const kmq::GemmArgs a{W, codebook, X, Y, N, K, M, bits, layout, workspace, workspace_bytes, scales};
    return kmq::check_and_run(a, hip_stream);
}

kmq_status kmq_gemv_blockscaled(const uint32_t* W, const uint16_t* codebook, const uint16_t* scales,
                                const uint16_t* x, uint16_t* y, int64_t N, int64_t K, int bits, int layout,
                                void* workspace, size_t workspace_bytes, void* hip_stream) {
    return kmq_gemm_smallbatch_blockscaled(W, codebook, scales, x, y, N, K, 1, bits, layout, workspace,
                                           workspace_bytes, hip_stream);
}

const char* kmq_kernel_name_blockscaled(int64_t N, int64_t K, int bits, int M, int layout) {
    return kmq::make_plan(N, K, bits, M, layout, true).name;
}

kmq_status kmq_dequant(const uint32_t* W, const uint16_t* codebook, uint16_t* Wdense,
                       int64_t N, int64_t K, int bits, int layout, void* hip_stream) {
    if (!W || !codebook || !Wdense) return KMQ_ERR_NULL;
    if (!kmq::bits_valid(bits)) return KMQ_ERR_BITS;
    if (!kmq::dims_valid(N, K)) return KMQ_ERR_SHAPE;
    if (layout != KMQ_LAYOUT_CANONICAL && layout != KMQ_LAYOUT_TILED) return KMQ_ERR_LAYOUT;
    if (layout == KMQ_LAYOUT_TILED && !kmq::tiled_valid(bits, K)) return KMQ_ERR_LAYOUT;
    if ((reinterpret_cast<uintptr_t>(W) & 15) || (reinterpret_cast<uintptr_t>(codebook) & 3) ||
        (reinterpret_cast<uintptr_t>(Wdense) & 1)) return KMQ_ERR_ALIGN;
    const hipError_t e = kmq::launch_dequant(W, codebook, Wdense, N, K, bits, layout,
                                             static_cast<hipStream_t>(hip_stream));
    return kmq::hip_status(e);
}

kmq_status kmq_gemv_bf16(const uint16_t* W, const uint16_t* x, uint16_t* y, int64_t N, int64_t K,
                         void* hip_stream) {
    if (!W || !x || !y) return KMQ_ERR_NULL;
    if (!kmq::dims_valid(N, K) || K > 32768) return KMQ_ERR_SHAPE;
    const uintptr_t a = (K % 8) == 0 ? 15 : 1;
    if ((reinterpret_cast<uintptr_t>(W) & a) || (reinterpret_cast<uintptr_t>(x) & a) ||
        (reinterpret_cast<uintptr_t>(y) & 1)) return KMQ_ERR_ALIGN;
    return kmq::hip_status(kmq::launch_gemv_bf16(W, x, y, N, K, static_cast<hipStream_t>(hip_stream)));
}

kmq_status kmq_quantize_rows(const uint16_t* Wdense, int64_t N, int64_t K, int bits, int iters,
                             uint32_t* packed, uint16_t* codebook, void* hip_stream) {
    if (!Wdense || !packed || !codebook) return KMQ_ERR_NULL;
    if (!kmq::bits_valid(bits) || bits > 4) return KMQ_ERR_BITS;
    if (!kmq::dims_valid(N, K) || iters < 0 || N > 0x7FFFFFFF) return KMQ_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(Wdense) & 1) || (reinterpret_cast<uintptr_t>(codebook) & 1) ||
        (reinterpret_cast<uintptr_t>(packed) & 3)) return KMQ_ERR_ALIGN;
    return kmq::hip_status(kmq::launch_quantize_rows(Wdense, N, K, bits, iters, packed, codebook,
                                                     static_cast<hipStream_t>(hip_stream)));
}

size_t kmq_quantize_blockscaled_workspace_bytes(void) { return kmq::quantize_blockscaled_workspace_bytes(); }

kmq_status kmq_quantize_blockscaled(const uint16_t* Wdense, int64_t N, int64_t K, int bits, int iters,
                                    uint32_t* packed, uint16_t* codebook, uint16_t* scales,
                                    void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!Wdense || !packed || !codebook || !scales) return KMQ_ERR_NULL;
    if (!kmq::bits_valid(bits) || bits > 4) return KMQ_ERR_BITS;
    if (!kmq::dims_valid(N, K) || iters < 0 || K % KMQ_BLOCK != 0 || N * (K / KMQ_BLOCK) > (int64_t(1) << 32))
        return KMQ_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(Wdense) & 15) || (reinterpret_cast<uintptr_t>(codebook) & 1) ||
        (reinterpret_cast<uintptr_t>(scales) & 1) || (reinterpret_cast<uintptr_t>(packed) & 3) ||
        (reinterpret_cast<uintptr_t>(workspace) & 7)) return KMQ_ERR_ALIGN;
    if (!workspace || workspace_bytes < kmq::quantize_blockscaled_workspace_bytes()) return KMQ_ERR_WORKSPACE;
    return kmq::hip_status(kmq::launch_quantize_blockscaled(Wdense, N, K, bits, iters, packed, codebook, scales,
                                                            workspace, static_cast<hipStream_t>(hip_stream)));
}

kmq_status kmq_dequant_blockscaled(const uint32_t* W, const uint16_t* codebook, const uint16_t* scales,
                                   uint16_t* Wdense, int64_t N, int64_t K, int bits, void* hip_stream) {
    if (!W || !codebook || !scales || !Wdense) return KMQ_ERR_NULL;
    if (!kmq::bits_valid(bits)) return KMQ_ERR_BITS;
    if (!kmq::dims_valid(N, K) || K % KMQ_BLOCK != 0 || N * (K / 8) > (int64_t(1) << 39)) return KMQ_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(W) & 15) || (reinterpret_cast<uintptr_t>(codebook) & 3) ||
        (reinterpret_cast<uintptr_t>(scales) & 1) || (reinterpret_cast<uintptr_t>(Wdense) & 15)) return KMQ_ERR_ALIGN;
    return kmq::hip_status(kmq::launch_dequant_blockscaled(W, codebook, scales, Wdense, N, K, bits,
                                                           static_cast<hipStream_t>(hip_stream)));
}

const char* kmq_last_hip_error(void) { return kmq::g_last_hip_error; }

}  // extern "C"
