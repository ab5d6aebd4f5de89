// Shard products: C_s = op(A_s) op(B_s) for all shards in one launch (Sec. 5.2 step 2 of arXiv 1805.04170:
// after input conversion every device runs the same sub-operator on its own tiles).
//
// bf16 path: the MFMA tile engine of gemm_core.h with dense-matrix loaders (NN, NT, TN, TT all share one main loop).
// fp32, rows without 16-byte vectors or off 16-byte boundaries, operands of 2^31 elements and more: gemm_small.hip.
#include "tt_device.h"
#include <cstdint>
#include <cstdlib>
#include <type_traits>
#include "gemm_core.h"
#include "gemm_core2.h"
#include "tt_internal.h"
#include "launch_util.h"

namespace tt {
namespace {

using core::kXcds;

template <int NS, int NC> struct GemmParamsT { // tables of NS shards and NC outputs
    const void *A[NS];
    const void *B[NS];
    void *C[NC];
    int32_t M, N, K;
    int32_t lda, ldb, ldc;
    int32_t tiles_m, tiles_n;
    int32_t per_xcd;  // logical workgroups per XCD (grid = per_xcd * 8)
    int32_t total;    // tiles_m * tiles_n * count * ksplit
    int32_t relu;
    int32_t nts;      // non-temporal stores (the engines of gemm_mma.h)
    int32_t ksplit;   // each shard's K range is cut into ksplit chunks of kchunk (a multiple of 64); chunk c of shard s
    int32_t kchunk;   // writes its own output C[s * ksplit + c] (partial sums, added up by the reduction kernel)
};
using GemmParams = GemmParamsT<kMaxShards, kMaxShards>;

template <int BM, int BN, int WM, int WN, int DEPTH, bool KMASK, bool A_KC, bool B_KC, bool OUT_BF16, bool VEC, class P>
__device__ __forceinline__ void run_bf16_tile(const P &p, int logical, uint16_t *smem)
{
    const int tiles = p.tiles_m * p.tiles_n;
    const int vshard = logical / tiles;
    const int t = logical - vshard * tiles;
    int tm, tn;
    core::grouped_tile(t, p.tiles_m, p.tiles_n, &tm, &tn);
    const int shard = vshard / p.ksplit;
    const int kbeg = (vshard - shard * p.ksplit) * p.kchunk;
    const int klen = p.K - kbeg < p.kchunk ? p.K - kbeg : p.kchunk;

    constexpr int NT = WM * WN * 64;
    constexpr int SA = core::Slots<BM, A_KC, NT>::value, SB = core::Slots<BN, B_KC, NT>::value;
    using LA = std::conditional_t<A_KC, core::DenseKC<SA>, core::DenseRC<SA>>;
    using LB = std::conditional_t<B_KC, core::DenseKC<SB>, core::DenseRC<SB>>;
    LA la;
    la.base = reinterpret_cast<const char *>(p.A[shard]) + (size_t)kbeg * (A_KC ? 2 : 2 * (size_t)p.lda);
    la.ld = p.lda; la.rows = p.M; la.K = klen;
    LB lb;
    lb.base = reinterpret_cast<const char *>(p.B[shard]) + (size_t)kbeg * (B_KC ? 2 : 2 * (size_t)p.ldb);
    lb.ld = p.ldb; lb.rows = p.N; lb.K = klen;
    core::tile_product<BM, BN, WM, WN, DEPTH, KMASK, OUT_BF16, VEC>(la, lb, p.C[vshard], p.ldc, p.M, p.N, klen, tm * BM, tn * BN, p.relu != 0, smem);
}

template <int BM, int BN, int WM, int WN, int DEPTH, bool KMASK, bool A_KC, bool B_KC, bool OUT_BF16, bool VEC>
__global__ __launch_bounds__(WM * WN * 64, WM * WN / 4) void gemm_bf16_kernel(const GemmParams p)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    const int logical = core::logical_block(p.per_xcd, p.total);
    if (logical < 0) return;
    run_bf16_tile<BM, BN, WM, WN, DEPTH, KMASK, A_KC, B_KC, OUT_BF16, VEC>(p, logical, smem);
}

// A B^T (DM x 128 tiles) and A^T B (128 x 128) of a backward step in one launch
struct GemmPair {
    GemmParamsT<8, 64> dgrad;
    GemmParamsT<8, 8> wgrad;
};
template <int DM, bool KMASK, bool D_BF16> __global__ __launch_bounds__(256, 2) void gemm_bf16_pair_kernel(const GemmPair p)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    const int first = p.dgrad.per_xcd * kXcds, bid = (int)blockIdx.x; // (a multiple of the XCDs: both parts are dealt out alike)
    if (bid < first) {
        const int logical = core::logical_block(bid, p.dgrad.per_xcd, p.dgrad.total);
        if (logical < 0) return;
        constexpr int WM = DM == 128 ? 2 : 1, DEPTH = DM == 128 ? 1 : 2;
        run_bf16_tile<DM, 128, WM, 4 / WM, DEPTH, KMASK, true, true, D_BF16, true>(p.dgrad, logical, smem);
    } else {
        const int logical = core::logical_block(bid - first, p.wgrad.per_xcd, p.wgrad.total);
        if (logical < 0) return;
        run_bf16_tile<128, 128, 2, 2, 1, KMASK, false, false, true, true>(p.wgrad, logical, smem);
    }
}
template <int DM, bool KMASK, bool D_BF16> tt_status launch_bf16_pair(const GemmPair &p, hipStream_t s)
{
    auto kern = gemm_bf16_pair_kernel<DM, KMASK, D_BF16>;
    constexpr size_t d = core::smem_bytes<DM, 128, DM == 128 ? 1 : 2>(), w = core::smem_bytes<128, 128, 1>(), smem = d > w ? d : w;
    if (ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem) != TT_OK) return TT_EDEVICE;
    hipLaunchKernelGGL(kern, dim3((uint32_t)(p.dgrad.per_xcd + p.wgrad.per_xcd) * kXcds), dim3(256), smem, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}
template <bool KMASK> tt_status launch_bf16_pair_rows(const GemmPair &p, int DM, bool d_bf16, hipStream_t s)
{
    if (DM == 32) return d_bf16 ? launch_bf16_pair<32, KMASK, true>(p, s) : launch_bf16_pair<32, KMASK, false>(p, s);
    if (DM == 64) return d_bf16 ? launch_bf16_pair<64, KMASK, true>(p, s) : launch_bf16_pair<64, KMASK, false>(p, s);
    return d_bf16 ? launch_bf16_pair<128, KMASK, true>(p, s) : launch_bf16_pair<128, KMASK, false>(p, s);
}

// second engine: operand tiles loaded straight into LDS, 256 x 256 tiles, eight waves
template <bool A_KC, bool B_KC, bool OUT_BF16, bool VEC>
__global__ __launch_bounds__(core2::kThreads2, 2) void gemm_bf16_v2_kernel(const GemmParams p)
{
    extern __shared__ __attribute__((aligned(16))) char smem2[];
    const int logical = core::logical_block(p.per_xcd, p.total);
    if (logical < 0) return;
    const int tiles = p.tiles_m * p.tiles_n;
    const int vshard = logical / tiles;
    const int t = logical - vshard * tiles;
    int tm, tn;
    core::grouped_tile(t, p.tiles_m, p.tiles_n, &tm, &tn);
    const int shard = vshard / p.ksplit;
    const int kbeg = (vshard - shard * p.ksplit) * p.kchunk;
    const int klen = p.K - kbeg < p.kchunk ? p.K - kbeg : p.kchunk;
    using LA = std::conditional_t<A_KC, core2::DenseKC2, core2::DenseRC2>;
    using LB = std::conditional_t<B_KC, core2::DenseKC2, core2::DenseRC2>;
    LA la;
    la.base = reinterpret_cast<const char *>(p.A[shard]) + (size_t)kbeg * (A_KC ? 2 : 2 * (size_t)p.lda);
    la.ld = p.lda; la.rows = p.M; la.K = klen;
    LB lb;
    lb.base = reinterpret_cast<const char *>(p.B[shard]) + (size_t)kbeg * (B_KC ? 2 : 2 * (size_t)p.ldb);
    lb.ld = p.ldb; lb.rows = p.N; lb.K = klen;
    core2::tile_product2<OUT_BF16, VEC>(la, lb, p.C[vshard], p.ldc, p.M, p.N, klen, tm * 256, tn * 256, p.relu != 0, smem2, p.nts != 0);
}

template <bool A_KC, bool B_KC, bool OUT_BF16, bool VEC> tt_status launch_v2(GemmParams &p, int count, hipStream_t s)
{
    auto kern = gemm_bf16_v2_kernel<A_KC, B_KC, OUT_BF16, VEC>;
    if (ensure_dynamic_lds(reinterpret_cast<const void *>(kern), core2::kSmemBytes) != TT_OK) return TT_EDEVICE;
    p.tiles_m = (p.M + 255) / 256;
    p.tiles_n = (p.N + 255) / 256;
    int64_t total = (int64_t)p.tiles_m * p.tiles_n * count * p.ksplit;
    if (total >= (int64_t(1) << 30)) return TT_EUNSUPPORTED;
    p.total = (int32_t)total;
    p.per_xcd = (int32_t)((total + kXcds - 1) / kXcds);
    hipLaunchKernelGGL(kern, dim3((uint32_t)p.per_xcd * kXcds), dim3(core2::kThreads2), core2::kSmemBytes, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

// BM x 128 tiles straight into LDS, four waves, three stages of 64 (72 KB for 64 rows: two workgroups per CU)
constexpr int kRowsStages = 3;
template <int BM, bool A_KC, bool B_KC, bool OUT_BF16, bool VEC>
__global__ __launch_bounds__(core::kThreads, 2) void gemm_bf16_rows_kernel(const GemmParams p)
{
    extern __shared__ __attribute__((aligned(16))) char smem2[];
    const int logical = core::logical_block(p.per_xcd, p.total);
    if (logical < 0) return;
    const int tiles = p.tiles_m * p.tiles_n;
    const int vshard = logical / tiles;
    const int t = logical - vshard * tiles;
    int tm, tn;
    core::grouped_tile(t, p.tiles_m, p.tiles_n, &tm, &tn);
    const int shard = vshard / p.ksplit;
    const int kbeg = (vshard - shard * p.ksplit) * p.kchunk;
    const int klen = p.K - kbeg < p.kchunk ? p.K - kbeg : p.kchunk;
    using LA = std::conditional_t<A_KC, core2::DenseKCT<core::kThreads>, core2::DenseRCT<core::kThreads>>;
    using LB = std::conditional_t<B_KC, core2::DenseKCT<core::kThreads>, core2::DenseRCT<core::kThreads>>;
    LA la;
    la.base = reinterpret_cast<const char *>(p.A[shard]) + (size_t)kbeg * (A_KC ? 2 : 2 * (size_t)p.lda);
    la.ld = p.lda; la.rows = p.M; la.K = klen;
    LB lb;
    lb.base = reinterpret_cast<const char *>(p.B[shard]) + (size_t)kbeg * (B_KC ? 2 : 2 * (size_t)p.ldb);
    lb.ld = p.ldb; lb.rows = p.N; lb.K = klen;
    core2::tile_product<OUT_BF16, VEC, BM, 128, 2, 2, kRowsStages>(la, lb, p.C[vshard], p.ldc, p.M, p.N, klen, tm * BM, tn * 128, p.relu != 0, smem2, p.nts != 0);
}

template <int BM, bool A_KC, bool B_KC, bool OUT_BF16, bool VEC> tt_status launch_rows_cfg(GemmParams &p, int count, hipStream_t s)
{
    auto kern = gemm_bf16_rows_kernel<BM, A_KC, B_KC, OUT_BF16, VEC>;
    constexpr size_t smem = (size_t)kRowsStages * (BM + 128) * core::BK * 2;
    if (ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem) != TT_OK) return TT_EDEVICE;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + 127) / 128;
    const int64_t total = (int64_t)p.tiles_m * p.tiles_n * count * p.ksplit;
    if (total >= (int64_t(1) << 30)) return TT_EUNSUPPORTED;
    p.total = (int32_t)total;
    p.per_xcd = (int32_t)((total + kXcds - 1) / kXcds);
    hipLaunchKernelGGL(kern, dim3((uint32_t)p.per_xcd * kXcds), dim3(core::kThreads), smem, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

template <int BM, int BN, int WM, int WN, int DEPTH, bool KMASK, bool A_KC, bool B_KC, bool OUT_BF16, bool VEC>
tt_status launch_mfma_cfg(GemmParams &p, int count, hipStream_t s)
{
    auto kern = gemm_bf16_kernel<BM, BN, WM, WN, DEPTH, KMASK, A_KC, B_KC, OUT_BF16, VEC>;
    constexpr size_t smem = core::smem_bytes<BM, BN, DEPTH>();
    if (ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem) != TT_OK) return TT_EDEVICE;
    p.tiles_m = (p.M + BM - 1) / BM;
    p.tiles_n = (p.N + BN - 1) / BN;
    int64_t total = (int64_t)p.tiles_m * p.tiles_n * count * p.ksplit;
    if (total >= (int64_t(1) << 30)) return TT_EUNSUPPORTED;
    p.total = (int32_t)total;
    p.per_xcd = (int32_t)((total + kXcds - 1) / kXcds);
    hipLaunchKernelGGL(kern, dim3((uint32_t)p.per_xcd * kXcds), dim3(WM * WN * 64), smem, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

// Tile choice (TT_GEMM_TILE overrides; tuning aid).
//   5: 256 x 256, whenever the launch has enough tiles to put work on at least half the CUs: the large tile halves operand
//      traffic per flop.  (The persistent engine, or gemm_core2.h.)
//   0: 256 x 128, four waves, two K tiles prefetched in registers: long K loops with few column tiles.
//   1: 128 x 128, four waves, up to two workgroups per CU: small products and short K loops.
//   8 (forced only): 256 x 256 on gemm_core2.h.
int pick_tile(int64_t M, int64_t N, int64_t K, int count)
{
    const int forced = tuning_int("TT_GEMM_TILE", -1);
    if (forced == 0 || forced == 1 || forced == 5 || forced == 8) return forced;
    const int64_t big = ((M + 255) / 256) * ((N + 255) / 256) * count;
    if (M > 128 && N > 128 && big >= 128) return 5;
    return (M > 128 && K >= 1024) ? 0 : 1;
}

// 128 x 128 tiles: whether a second K tile on its way pays.  At most one workgroup per CU: its registers are free for it.
// At least three K tiles: with one or two the wider prologue costs 0.2-0.5 us of 5.  Full column tiles: where the last
// one is short, one tile ahead already runs faster (fewer lanes load) and two lose 0.5-1.5 us; with A row-contiguous only
// where rows are cut short too, up to K of about 768.  One tile ahead / two, us: 16 x (128 x 128) NN K 64 4.7 / 4.8, 320 7.8 / 7.4, 1000
// 19.3 / 17.5, TN 320 9.7 / 9.1, 1000 24.0 / 19.0;  4 x (200 x 264) NN 264 7.7 / 8.4, 1000 16.2 / 17.7, TN 264 8.1 / 8.5;  8 x (128 x 264) TN
// 264 8.8 / 8.5, 1000 20.9 / 17.5;  16 x (40 x 40) TN 320 7.7 / 8.0, 1000 17.5 / 17.7.
bool two_tiles_ahead(int64_t M, int64_t N, int64_t K, int64_t outs, bool a_kc)
{
    const int64_t tiles_n = (N + 127) / 128;
    if ((M + 127) / 128 * tiles_n * outs > 256 || K <= 128) return false;
    if (N % 128 == 0) return true;
    return !a_kc && (M % 128 == 0 || (tiles_n * 128 - N) * 16 <= N || K >= 768);
}

// Products with at most 128 rows whose tiles go straight into LDS, and their rows per tile (0: through registers).  What these
// products wait for is memory: two K tiles on their way without a register hop, and, for 65 to 128 rows, twice as many
// workgroups on half the rows each while two of them per CU hold all tiles.  Through registers / so, two shards, us:
// 128 x 1024 A B^T K 512 9.3 / 8.0, 1024 14.2 / 11.5, 2048 23.7 / 18.9, x 16384 (512 tiles) 11.3 / 10.8, 18.6 / 20.1, 38.0 / 42.1;
// A B the same (2048: 26.5 / 21.6); 8 x (72 x 1176 x 4640) A B^T 97 / 43.  Fewer rows: A B of long K only: 32 x 1024 K 512 7.2 /
// 7.9, 1024 11.9 / 11.4, 2048 20.2 / 19.3, x 16384 14.6 / 13.5, 29.5 / 24.3 (32 rows); 48 x 1024 K 1024 12.0 / 12.9, 2048 22.6 / 21.5, x 16384
// 31.0 / 24.5 (64 rows); A B^T 32 x 1024 K 2048 14.8 / 15.4.
int rows_into_lds(int64_t M, int64_t N, int64_t K, int64_t outs, bool b_kc)
{
    if (M > 128) return 0;
    if (M > 64) return K >= 384 && (N + 127) / 128 * 2 * outs < 512 ? 64 : 0;
    if (b_kc) return 0;
    return M > 32 ? (K >= 2048 ? 64 : 0) : (K >= 1024 ? 32 : 0);
}

template <bool KMASK, bool A_KC, bool B_KC, bool OUT_BF16, bool VEC> tt_status launch_mfma_tile(GemmParams &p, int count, hipStream_t s)
{
    const int tile = pick_tile(p.M, p.N, p.ksplit > 1 ? p.kchunk : p.K, count * p.ksplit);
    if (tile == 0) return launch_mfma_cfg<256, 128, 2, 2, 2, KMASK, A_KC, B_KC, OUT_BF16, VEC>(p, count, s);
    if (tuning_int("TT_GEMM_TILE", -1) < 0) {
        // Few rows (a small batch against streamed weights): a 128-row tile would take in, store to LDS and multiply rows that
        // do not exist; what counts is how much of the weights is on its way, and the narrower tiles have two K tiles of
        // it in registers and several workgroups per CU.  8 x (16 x 4096 x 1152) 29.2 -> 19.4 us, 8 x (8 x 4096 x 9216) 189 -> 120
        // (5 TB/s of weights), 64 x 4096 x 4096 68 -> 42 us.  (32 rows: A K-contiguous only, its loader needs a chunk per thread.)
        if constexpr (A_KC) {
            if (p.M <= 32) return launch_mfma_cfg<32, 128, 1, 4, 2, KMASK, A_KC, B_KC, OUT_BF16, VEC>(p, count, s);
            if (p.M <= 64) return launch_mfma_cfg<64, 128, 1, 4, 2, KMASK, A_KC, B_KC, OUT_BF16, VEC>(p, count, s);
        }
        if (two_tiles_ahead(p.M, p.N, p.ksplit > 1 ? p.kchunk : p.K, count * p.ksplit, A_KC))
            return launch_mfma_cfg<128, 128, 2, 2, 2, KMASK, A_KC, B_KC, OUT_BF16, VEC>(p, count, s);
    }
    return launch_mfma_cfg<128, 128, 2, 2, 1, KMASK, A_KC, B_KC, OUT_BF16, VEC>(p, count, s);
}

template <bool A_KC, bool B_KC, bool OUT_BF16, bool VEC> tt_status launch_mfma_kmask(GemmParams &p, int count, hipStream_t s)
{
    // Where the eight-wave 256 x 256 tile is chosen, the engine that loads tiles straight into LDS is the faster one (through
    // registers / into LDS, us: A B 2048 x 8200 x 4104 260 / 210, 4 x (1000 x 4000 x 1000) 42 / 35)
    const int tile = pick_tile(p.M, p.N, p.ksplit > 1 ? p.kchunk : p.K, count * p.ksplit);
    if constexpr (A_KC) {
        const int rows = tuning_int("TT_GEMM_TILE", -1) < 0 ? rows_into_lds(p.M, p.N, p.ksplit > 1 ? p.kchunk : p.K, count * p.ksplit, B_KC) : 0;
        if constexpr (!B_KC)
            if (rows == 32) return launch_rows_cfg<32, A_KC, B_KC, OUT_BF16, VEC>(p, count, s);
        if (rows == 64) return launch_rows_cfg<64, A_KC, B_KC, OUT_BF16, VEC>(p, count, s);
    }
    if ((tile == 8 || tile == 5) && p.M >= 8 && p.N >= 8) // (chosen, 5 has far more; forced, it may not)
        return launch_v2<A_KC, B_KC, OUT_BF16, VEC>(p, count, s);
    return p.K % core::BK ? launch_mfma_tile<true, A_KC, B_KC, OUT_BF16, VEC>(p, count, s)
                          : launch_mfma_tile<false, A_KC, B_KC, OUT_BF16, VEC>(p, count, s);
}

template <bool A_KC, bool B_KC> tt_status launch_mfma_out(GemmParams &p, int count, int out_dtype, int act, bool vec, hipStream_t s)
{
    p.relu = act == TT_ACT_RELU;
    if (out_dtype == TT_BF16)
        return vec ? launch_mfma_kmask<A_KC, B_KC, true, true>(p, count, s) : launch_mfma_kmask<A_KC, B_KC, true, false>(p, count, s);
    return vec ? launch_mfma_kmask<A_KC, B_KC, false, true>(p, count, s) : launch_mfma_kmask<A_KC, B_KC, false, false>(p, count, s);
}

bool all_aligned16(const void *const *ptrs, int n)
{
    for (int i = 0; i < n; ++i)
        if (reinterpret_cast<uintptr_t>(ptrs[i]) & 15) return false;
    return true;
}

// 16-byte vectors along each operand's contiguous side, byte offsets in 31 bits
bool mfma_takes(int count, const void *const *A, const void *const *B, int64_t M, int64_t N, int64_t K, bool trans_a, bool trans_b, int in_dtype)
{
    return in_dtype == TT_BF16 && K > 0 && (trans_a ? M : K) % 8 == 0 && (trans_b ? K : N) % 8 == 0 && M * K < (int64_t(1) << 31) &&
           K * N < (int64_t(1) << 31) && all_aligned16(A, count) && all_aligned16(B, count);
}

} // namespace

tt_status launch_gemm(int count, const void *const *A, const void *const *B, void *const *C, int64_t M, int64_t N,
                      int64_t K, int trans_a, int trans_b, int in_dtype, int out_dtype, int act, int ksplit, void *stream)
{
    if (!A || !B || !C || count < 0 || count > kMaxShards || M < 0 || N < 0 || K < 0) return TT_EINVAL;
    if ((in_dtype != TT_BF16 && in_dtype != TT_F32) || (out_dtype != TT_BF16 && out_dtype != TT_F32)) return TT_EINVAL;
    if (act != TT_ACT_NONE && act != TT_ACT_RELU) return TT_EINVAL;
    if (ksplit < 1 || count * ksplit > kMaxShards) return TT_EINVAL;
    if (count == 0 || M == 0 || N == 0) return TT_OK;
    if (M >= (int64_t(1) << 31) || N >= (int64_t(1) << 31) || K >= (int64_t(1) << 31)) return TT_EUNSUPPORTED;
    for (int s = 0; s < count; ++s)
        if (!A[s] || !B[s]) return TT_EINVAL;
    for (int s = 0; s < count * ksplit; ++s)
        if (!C[s]) return TT_EINVAL;
    // K chunk per split: a multiple of the tile depth; every chunk must be non-empty
    const int64_t kchunk = ksplit == 1 ? (K > 0 ? K : 1) : ((K + ksplit - 1) / ksplit + 63) / 64 * 64;
    if (ksplit > 1 && kchunk * (ksplit - 1) >= K) return TT_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);

    // MFMA path needs 16-byte vectors along each operand's contiguous dimension
    const int64_t a_contig = trans_a ? M : K, b_contig = trans_b ? K : N;
    // (operand byte offsets are kept in 32 bits inside the kernel)
    const bool mfma_ok = mfma_takes(count, A, B, M, N, K, trans_a != 0, trans_b != 0, in_dtype);
    const uint64_t in_b = in_dtype == TT_BF16 ? 2 : 4, out_b = out_dtype == TT_BF16 ? 2 : 4;
    const int kclass = !mfma_ok ? TT_K_GEMM_GENERIC
                                : (trans_a ? (trans_b ? TT_K_GEMM_TT : TT_K_GEMM_TN) : (trans_b ? TT_K_GEMM_NT : TT_K_GEMM_NN));
    ProfileScope scope(stream, kclass, count, M, N, K,
                       (uint64_t)count * (in_b * ((uint64_t)M * K + (uint64_t)K * N) + out_b * (uint64_t)M * N),
                       2ull * (uint64_t)M * (uint64_t)N * (uint64_t)K * (uint64_t)count);
    if (mfma_ok) {
        GemmParams p;
        for (int i = 0; i < kMaxShards; ++i) {
            p.A[i] = i < count ? A[i] : nullptr;
            p.B[i] = i < count ? B[i] : nullptr;
            p.C[i] = i < count * ksplit ? C[i] : nullptr;
        }
        p.M = (int32_t)M; p.N = (int32_t)N; p.K = (int32_t)K;
        p.lda = (int32_t)a_contig;
        p.ldb = (int32_t)b_contig;
        p.ldc = (int32_t)N;
        p.nts = non_temporal_results(N * (int64_t)out_b, M * N * (int64_t)out_b * count * ksplit);
        p.ksplit = ksplit;
        p.kchunk = (int32_t)kchunk;
        const bool a_kc = !trans_a, b_kc = trans_b != 0;
        // 16-byte stores along C's rows need 16-byte row pitch and base addresses
        const bool vec = N % (out_dtype == TT_BF16 ? 8 : 4) == 0 && all_aligned16(const_cast<const void *const *>(C), count * ksplit);
        // Engine choice (TT_GEMM_ENGINE=1: the two older engines only, =3 / =4: that engine wherever it applies; tuning aid):
        //  - launches with too few 256 x 256 tiles to occupy the chip (the hidden-layer products at batch 256): the
        //    256 x 128 engine with two workgroups per CU, which doubles the number of workgroups;
        //  - larger launches: the persistent pipelined engine where K is a multiple of 64 (16 x (256 x 4096 x 640) A^T B 26.9 -> 25.1 us
        //    against the direct-to-LDS engine, A B^T over K = 512 28.3 -> 28.0), else the direct-to-LDS engine.
        const int engine = tuning_int("TT_GEMM_ENGINE", 0);
        const int64_t big_tiles = ((M + 255) / 256) * ((N + 255) / 256) * count * ksplit;
        //  - weight-gradient shaped products (both operands stored with K as the slow dimension, K up to 256 or 512, a bf16
        //    result large enough to give every resident workgroup at least two 256 x 64 units; measured down to the second
        //    VGG-16 weight gradient, 8 x 1024 x 2048 x 256: 16 us against 20 us on the persistent engine): the engine that
        //    keeps the left operand's panel in registers and is bound by writing the result (gemm_core5.h).  Any K up to 256 runs
        //    on the next of 64, 128 and 256, between 256 and 512 the padding costs more than it saves.  Here / 256 x 128 tiles / the
        //    larger ones, us: 6936 x 7456 K 219 38 / 44 / 57, K 300 66 / 51 / 62, K 480 69 / 60 / 82; 13504 x 4288 K 72 31 / 32 / 41;
        //    9072 x 11856 K 40 86 / 103 / 91; 8 x (1568 x 4096) K 192 38 / 35 / 44
        if ((engine == 5 || engine == 0) && !a_kc && !b_kc && ksplit == 1 && out_dtype == TT_BF16 && vec && in_dtype == TT_BF16 &&
            (engine == 5 || (((M + 255) / 256) * ((N + 63) / 64) * count >= 2 * 512 && (K <= 256 || K == 512)))) {
            const tt_status st = launch_gemm_v5(count, A, B, C, M, N, K, a_contig, b_contig, N, act == TT_ACT_RELU, stream);
            if (st != TT_EUNSUPPORTED) return st;
        }
        //  - of those, launches of at most one 256 x 128 tile per CU and a K that is long enough for a start that fetches three stages
        //    of 48 KB: the same tile with K tiles of 64 and one workgroup per CU (gemm_core6.h).  gemm_core4.h / gemm_core6.h, eight
        //    shards of 256 rows, us: A B^T to 4096 columns K 256 9.2 / 9.6, 512 13.2 / 12.4, 1024 27.7 / 21.8, 2048 52.5 / 43.3 (1024
        //    columns 7.4 / 8.3, 10.7 / 10.5, 16.5 / 15.2, 28.4 / 24.5); A B 11.2 / 12.0, 15.1 / 15.3, 28.4 / 23.3, 51.5 / 40.4; A^T B to
        //    2048 columns, K 2048 38.9 / 33.9, 8 x (512 x 512 x 1024) 16.6 / 17.3; 288 tiles of K 1024 A B^T 30.3 / 31.3.  Short last K tiles:
        //    A^T B 8 x (1024 x 1024) K 1032 25.5 / 27.0, 2056 38.0 / 39.9, 3000 54.8 / 53.2, 4104 70.6 / 70.4, fp32 4 x (1024 x 2048 x 2088) 44.0 /
        //    42.5; 8 x (256 x 2048) A B^T K 520 11.9 / 12.6, 1032 24.2 / 21.3, A B K 1032 21.2 / 21.1
        const int64_t kc = ksplit > 1 ? kchunk : K;
        const int64_t tiles128 = ((M + 255) / 256) * ((N + 127) / 128) * count * ksplit;
        if (engine == 6 || (engine == 0 && big_tiles < 200 && M > 128 && N >= 256 && tiles128 <= 256 &&
                                                   kc >= (!a_kc ? 2048 : b_kc ? 512 : 1024))) {
            const tt_status st = launch_gemm_v6(count, A, B, C, M, N, K, a_contig, b_contig, N, a_kc, b_kc, out_dtype, act == TT_ACT_RELU,
                                                vec, ksplit, kchunk, stream);
            if (st != TT_EUNSUPPORTED) return st;
        }
        //  - 256 x 128 tiles, two workgroups per CU, otherwise; K that is no multiple of 32 from 128 on (8 x (300 x 4000 x 200) A B through
        //    registers 14.4, here 11.6; K 104 6.2 / 7.7), but for A B^T where 256 x 256 tiles keep half the CUs busy and there are more of these
        //    than CUs (2 x (997 x 5144 x 1288) 52 here, 42 on the larger tile).  Of the larger launches those whose K the persistent engine does not take and
        //    that are short enough for the second workgroup to be worth the narrower tile.  Direct-to-LDS engine / here, us: A^T B 6936 x
        //    7456 K 529 84 / 67, 1001 128 / 114, 1529 178 / 163, 8 x (1936 x 832) K 16 10.1 / 8.6; 8 x (500 x 8000) A B K 200 28.7 / 24.1, 520 45.8 / 44.0,
        //    1032 73.9 / 90.4; A B^T K 200 28.9 / 26.8, 520 44.8 / 49.8
        const bool narrow = big_tiles < 200 ? K % 32 == 0 || (kc >= 128 && !(a_kc && b_kc && big_tiles >= 128 && tiles128 > 256))
                                            : K % 64 != 0 ? (!a_kc && !b_kc ? kc <= 2048 : kc >= 64 && kc <= (a_kc && !b_kc ? 640 : 256))
                                                          : !a_kc && !b_kc && kc > 256 && kc < 512;
        if (engine == 4 || (engine == 0 && narrow && M > 128 && N >= 256)) {
            const tt_status st = launch_gemm_v4(count, A, B, C, M, N, K, a_contig, b_contig, N, a_kc, b_kc, out_dtype,
                                                act == TT_ACT_RELU, vec, ksplit, kchunk, stream);
            if (st != TT_EUNSUPPORTED) return st;
        }
        if (engine != 1 && engine != 4 && pick_tile(M, N, ksplit > 1 ? kchunk : K, count * ksplit) == 5) {
            const tt_status st = launch_gemm_v3(count, A, B, C, M, N, K, a_contig, b_contig, N, a_kc, b_kc, out_dtype,
                                                act == TT_ACT_RELU, vec, ksplit, kchunk, stream);
            if (st != TT_EUNSUPPORTED) return st;
        }
        if (a_kc && b_kc) return launch_mfma_out<true, true>(p, count, out_dtype, act, vec, s);
        if (a_kc && !b_kc) return launch_mfma_out<true, false>(p, count, out_dtype, act, vec, s);
        if (!a_kc && !b_kc) return launch_mfma_out<false, false>(p, count, out_dtype, act, vec, s);
        return launch_mfma_out<false, true>(p, count, out_dtype, act, vec, s);
    }
    return launch_gemm_small(count, A, B, C, M, N, K, a_contig, b_contig, !trans_a, trans_b != 0, in_dtype, out_dtype,
                             act == TT_ACT_RELU, ksplit, kchunk, stream);
}

tt_status launch_gemm_runs(int nblk, int nred, int parts, const void *const *A, const void *const *B, void *const *C, int64_t M, int64_t N,
                           int64_t K, int trans_a, int trans_b, int out_dtype, int act, void *stream)
{
    if (!A || !B || !C || nblk < 1 || nred < 1 || parts < 1 || nblk * nred > kMaxShards || nblk * parts > kMaxShards) return TT_EUNSUPPORTED;
    if (M < 1 || N < 1 || K < 1 || M >= (int64_t(1) << 31) || N >= (int64_t(1) << 31) || K >= (int64_t(1) << 31)) return TT_EUNSUPPORTED;
    for (int i = 0; i < nblk * nred; ++i)
        if (!A[i] || !B[i]) return TT_EUNSUPPORTED;
    for (int i = 0; i < nblk * parts; ++i)
        if (!C[i]) return TT_EUNSUPPORTED;
    if (!mfma_takes(nblk * nred, A, B, M, N, K, trans_a != 0, trans_b != 0, TT_BF16)) return TT_EUNSUPPORTED;
    if (N % (out_dtype == TT_BF16 ? 8 : 4) || !all_aligned16(const_cast<const void *const *>(C), nblk * parts)) return TT_EUNSUPPORTED;
    return launch_gemm_v3_runs(nblk, nred, parts, A, B, C, M, N, K, trans_a ? M : K, trans_b ? K : N, N, !trans_a, trans_b != 0, out_dtype,
                               act == TT_ACT_RELU, stream);
}

namespace {

template <class P> void fill_pair_half(P *p, const GemmCall &c, bool dgrad, int BM, int ns, int nc)
{
    for (int i = 0; i < ns; ++i) {
        p->A[i] = i < c.count ? c.A[i] : nullptr;
        p->B[i] = i < c.count ? c.B[i] : nullptr;
    }
    for (int i = 0; i < nc; ++i) p->C[i] = i < c.count * c.ksplit ? c.C[i] : nullptr;
    p->M = (int32_t)c.M; p->N = (int32_t)c.N; p->K = (int32_t)c.K;
    p->lda = (int32_t)(dgrad ? c.K : c.M);
    p->ldb = (int32_t)(dgrad ? c.K : c.N);
    p->ldc = (int32_t)c.N;
    p->tiles_m = (int32_t)((c.M + BM - 1) / BM);
    p->tiles_n = (int32_t)((c.N + 127) / 128);
    p->total = p->tiles_m * p->tiles_n * c.count * c.ksplit;
    p->per_xcd = (p->total + kXcds - 1) / kXcds;
    p->relu = 0;
    p->nts = 1;
    p->ksplit = c.ksplit;
    p->kchunk = (int32_t)(c.ksplit == 1 ? c.K : ((c.K + c.ksplit - 1) / c.ksplit + 63) / 64 * 64);
}

// Whether a result of one product lies over an operand of the other (a weight gradient stored in the place of the weights), or over
// a result: such products run one after the other.
bool in_each_other_s_way(const GemmCall &d, const GemmCall &w)
{
    const auto meet = [](const void *const *p, int np, uint64_t pb, const void *const *q, int nq, uint64_t qb) {
        for (int i = 0; i < np; ++i) {
            const uintptr_t a = reinterpret_cast<uintptr_t>(p[i]);
            for (int j = 0; j < nq; ++j) {
                const uintptr_t b = reinterpret_cast<uintptr_t>(q[j]);
                if (a < b + qb && b < a + pb) return true;
            }
        }
        return false;
    };
    const auto elem = [](int dtype) { return dtype == TT_BF16 ? uint64_t(2) : uint64_t(4); };
    const GemmCall *const g[2] = {&d, &w};
    uint64_t a[2], b[2], c[2];
    const void *const *out[2];
    for (int i = 0; i < 2; ++i) {
        a[i] = elem(g[i]->in_dtype) * (uint64_t)g[i]->M * (uint64_t)g[i]->K;
        b[i] = elem(g[i]->in_dtype) * (uint64_t)g[i]->K * (uint64_t)g[i]->N;
        c[i] = elem(g[i]->out_dtype) * (uint64_t)g[i]->M * (uint64_t)g[i]->N;
        out[i] = const_cast<const void *const *>(g[i]->C);
    }
    const int outs[2] = {d.count * d.ksplit, w.count * w.ksplit};
    for (int i = 0; i < 2; ++i)
        if (meet(out[i], outs[i], c[i], g[1 - i]->A, g[1 - i]->count, a[1 - i]) || meet(out[i], outs[i], c[i], g[1 - i]->B, g[1 - i]->count, b[1 - i])) return true;
    return meet(out[0], outs[0], c[0], out[1], outs[1], c[1]);
}

} // namespace

tt_status launch_gemm_pair(const GemmCall &d, const GemmCall &w, void *stream)
{
    const GemmCall *const g[2] = {&d, &w};
    bool mfma[2];
    for (int i = 0; i < 2; ++i) {
        const GemmCall &c = *g[i];
        if (!c.A || !c.B || !c.C || c.count < 1 || c.count > 8 || c.ksplit < 1 || c.count * c.ksplit > kMaxShards) return TT_EUNSUPPORTED;
        if (c.M < 1 || c.N < 1 || c.K < 1 || c.M >= (int64_t(1) << 31) || c.N >= (int64_t(1) << 31) || c.K >= (int64_t(1) << 31)) return TT_EUNSUPPORTED;
        for (int s = 0; s < c.count; ++s)
            if (!c.A[s] || !c.B[s]) return TT_EUNSUPPORTED;
        for (int s = 0; s < c.count * c.ksplit; ++s)
            if (!c.C[s]) return TT_EUNSUPPORTED;
        mfma[i] = mfma_takes(c.count, c.A, c.B, c.M, c.N, c.K, i == 1, i == 0, c.in_dtype);
    }
    if (mfma[0] != mfma[1] || in_each_other_s_way(d, w)) return TT_EUNSUPPORTED;
    if (!mfma[0]) return launch_ordered_pair(d, w, stream);
    // Results with 16-byte rows, the weight gradient in bf16 over K of at most 1024 (one K tile on its way, where a launch of its
    // own has two), and no more than two workgroups per CU of either on the 128-column tiles of the register-staged engine.
    // Backward call, apart / together, us: 256 x 4096-1000 on 8 shards 29.1 / 21.3, 256 x 512-512 on one 21.7 / 12.0, 64 x 1536-776 on 4
    // 16.4 / 9.7, 1024 x 1024-1024 on one 41.7 / 32.0, 128 x 4096-2048 on 8 (512 workgroups) 25.1 / 20.2.  (Two fit a CU: at the limit
    // the launch takes two rounds.)
    // Past that: 256 x 4096-4096 on 8 (1024) 43 / 51; 2048 x 512-512 on 8 (weight gradients over K = 2048) 47.9 / 54.1.
    if (w.ksplit != 1 || w.out_dtype != TT_BF16 || w.K > 1024) return TT_EUNSUPPORTED;
    if (w.N % 8 || d.N % (d.out_dtype == TT_BF16 ? 8 : 4) || !all_aligned16(const_cast<const void *const *>(w.C), w.count) ||
        !all_aligned16(const_cast<const void *const *>(d.C), d.count * d.ksplit))
        return TT_EUNSUPPORTED;
    const int DM = d.M <= 32 ? 32 : d.M <= 64 ? 64 : 128;
    static const int most = tuning_int("TT_PAIR_TILES", 512);
    if (((d.M + DM - 1) / DM) * ((d.N + 127) / 128) * d.count * d.ksplit > most || ((w.M + 127) / 128) * ((w.N + 127) / 128) * w.count > most)
        return TT_EUNSUPPORTED;
    GemmPair p;
    fill_pair_half(&p.dgrad, d, true, DM, 8, 64);
    fill_pair_half(&p.wgrad, w, false, 128, 8, 8);
    if (d.ksplit > 1 && (int64_t)p.dgrad.kchunk * (d.ksplit - 1) >= d.K) return TT_EUNSUPPORTED;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    ProfileScope scope(stream, TT_K_GEMM_PAIR, d.count, d.M, d.N, d.K, d.bytes() + w.bytes(), d.flops() + w.flops());
    return d.K % core::BK || w.K % core::BK ? launch_bf16_pair_rows<true>(p, DM, d.out_dtype == TT_BF16, s)
                                            : launch_bf16_pair_rows<false>(p, DM, d.out_dtype == TT_BF16, s);
}

} // namespace tt

extern "C" tt_status tt_shard_gemm(int count, const void *const *A, const void *const *B, void *const *C, int64_t M,
                                   int64_t N, int64_t K, int trans_a, int trans_b, int in_dtype, int out_dtype, int act,
                                   void *stream)
{
    return tt::launch_gemm(count, A, B, C, M, N, K, trans_a, trans_b, in_dtype, out_dtype, act, 1, stream);
}
