// Shard products on the persistent, software-pipelined MFMA engine (gemm_core3.h): kernels and launcher.
// One launch covers all shards (Sec. 5.2 step 2 of arXiv 1805.04170: every device runs the same sub-operator on its
// own tiles); the grid is one workgroup per CU and each workgroup walks its share of the 256 x 256 output tiles.
#include "tt_device.h"
#include <cstdint>
#include <cstdlib>
#include "gemm_core3.h"
#include "gemm_core4.h"
#include "gemm_core5.h"
#include "gemm_core6.h"
#include "gemm3_params.h"
#include "tt_internal.h"
#include "launch_util.h"

namespace tt {
namespace {

template <bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED, bool SPREAD, bool RUNS>
__global__ __launch_bounds__(core3::kThreads3, 2) void gemm_bf16_v3_kernel(const core3::Params3 p)
{
    extern __shared__ __attribute__((aligned(16))) char smem3[];
    core3::run_tiles<64, 2, A_KC, B_KC, OUT_BF16, STAGED, SPREAD, RUNS>(p, smem3);
}

// 256 x 128 tiles, four waves, two workgroups per CU (gemm_core4.h); one tile per workgroup
template <bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED, bool TAIL>
__global__ __launch_bounds__(core4::kThreads4, 2) void gemm_bf16_v4_kernel(const core3::Params3 p)
{
    extern __shared__ __attribute__((aligned(16))) char smem4[];
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
    const char *abase = reinterpret_cast<const char *>(p.A[shard]) + (size_t)kbeg * (A_KC ? 2 : 2 * (size_t)p.lda);
    const char *bbase = reinterpret_cast<const char *>(p.B[shard]) + (size_t)kbeg * (B_KC ? 2 : 2 * (size_t)p.ldb);
    core4::tile_product4<A_KC, B_KC, OUT_BF16, STAGED, TAIL>(abase, p.lda, bbase, p.ldb, p.C[vshard], p.ldc, p.M, p.N, klen,
                                                       tm * core4::BM4, tn * core4::BN4, p.relu != 0, smem4, p.nts != 0);
}

template <bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED, bool TAIL> tt_status launch_tail4(core3::Params3 &p, hipStream_t s)
{
    auto kern = gemm_bf16_v4_kernel<A_KC, B_KC, OUT_BF16, STAGED, TAIL>;
    if (ensure_dynamic_lds(reinterpret_cast<const void *>(kern), core4::kSmem4) != TT_OK) return TT_EDEVICE;
    hipLaunchKernelGGL(kern, dim3((uint32_t)p.per_xcd * core::kXcds), dim3(core4::kThreads4), core4::kSmem4, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

template <bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED> tt_status launch_cfg4(core3::Params3 &p, hipStream_t s)
{
    return p.K % core4::BK4 ? launch_tail4<A_KC, B_KC, OUT_BF16, STAGED, true>(p, s) : launch_tail4<A_KC, B_KC, OUT_BF16, STAGED, false>(p, s);
}

template <bool A_KC, bool B_KC> tt_status launch_layout4(core3::Params3 &p, int out_dtype, bool vec, hipStream_t s)
{
    const bool bf = out_dtype == TT_BF16;
    if (vec) return bf ? launch_cfg4<A_KC, B_KC, true, true>(p, s) : launch_cfg4<A_KC, B_KC, false, true>(p, s);
    return bf ? launch_cfg4<A_KC, B_KC, true, false>(p, s) : launch_cfg4<A_KC, B_KC, false, false>(p, s);
}

// 256 x 128 tiles, K tiles of 64, one workgroup per CU (gemm_core6.h); one tile per workgroup
template <bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED, bool TAIL>
__global__ __launch_bounds__(core6::kThreads6, 2) void gemm_bf16_v6_kernel(const core3::Params3 p)
{
    extern __shared__ __attribute__((aligned(16))) char smem4[];
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
    const char *abase = reinterpret_cast<const char *>(p.A[shard]) + (size_t)kbeg * (A_KC ? 2 : 2 * (size_t)p.lda);
    const char *bbase = reinterpret_cast<const char *>(p.B[shard]) + (size_t)kbeg * (B_KC ? 2 : 2 * (size_t)p.ldb);
    core6::tile_product6<A_KC, B_KC, OUT_BF16, STAGED, TAIL>(abase, p.lda, bbase, p.ldb, p.C[vshard], p.ldc, p.M, p.N, klen, tm * core6::BM6,
                                                       tn * core6::BN6, p.relu != 0, smem4, p.nts != 0);
}

template <bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED, bool TAIL> tt_status launch_tail6(core3::Params3 &p, hipStream_t s)
{
    auto kern = gemm_bf16_v6_kernel<A_KC, B_KC, OUT_BF16, STAGED, TAIL>;
    if (ensure_dynamic_lds(reinterpret_cast<const void *>(kern), core6::kSmem6) != TT_OK) return TT_EDEVICE;
    hipLaunchKernelGGL(kern, dim3((uint32_t)p.per_xcd * core::kXcds), dim3(core6::kThreads6), core6::kSmem6, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

template <bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED> tt_status launch_cfg6(core3::Params3 &p, hipStream_t s)
{
    return p.K % core6::BK6 ? launch_tail6<A_KC, B_KC, OUT_BF16, STAGED, true>(p, s) : launch_tail6<A_KC, B_KC, OUT_BF16, STAGED, false>(p, s);
}

template <bool A_KC, bool B_KC> tt_status launch_layout6(core3::Params3 &p, int out_dtype, bool vec, hipStream_t s)
{
    const bool bf = out_dtype == TT_BF16;
    if (vec) return bf ? launch_cfg6<A_KC, B_KC, true, true>(p, s) : launch_cfg6<A_KC, B_KC, false, true>(p, s);
    return bf ? launch_cfg6<A_KC, B_KC, true, false>(p, s) : launch_cfg6<A_KC, B_KC, false, false>(p, s);
}

// short-K products with the left operand's panel held in registers (gemm_core5.h); two workgroups per CU, one for KT = 32
template <int KT, bool NTS, bool TAIL> __global__ __launch_bounds__(core5::kThreads5, KT <= 16 ? 2 : 1) void gemm_bf16_v5_kernel(const core5::Params5 p)
{
    extern __shared__ __attribute__((aligned(16))) char smem3[];
    core5::run_panels<KT, NTS, TAIL>(p, smem3);
}

template <int KT, bool NTS, bool TAIL> tt_status launch_tail5(core5::Params5 &p, hipStream_t s)
{
    auto kern = gemm_bf16_v5_kernel<KT, NTS, TAIL>;
    constexpr size_t smem = core5::smem_bytes5<KT>();
    if (ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem) != TT_OK) return TT_EDEVICE;
    hipLaunchKernelGGL(kern, dim3((uint32_t)p.grid), dim3(core5::kThreads5), smem, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

template <int KT> tt_status launch_cfg5(core5::Params5 &p, hipStream_t s)
{
    // (rows that begin inside a 64-byte piece: see mma::store_block)
    const bool nts = p.ldc % 32 == 0;
    if (p.K == KT * 16) return nts ? launch_tail5<KT, true, false>(p, s) : launch_tail5<KT, false, false>(p, s);
    if constexpr (KT == 32 && !kTuning) return TT_EUNSUPPORTED; // (K between 256 and 512 goes elsewhere, launch_gemm)
    else return nts ? launch_tail5<KT, true, true>(p, s) : launch_tail5<KT, false, true>(p, s);
}

int cu_count()
{
    static const int n = [] {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 256;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
        return cus;
    }();
    return n;
}

template <bool A_KC, bool B_KC, bool OUT_BF16, bool STAGED, bool SPREAD, bool RUNS = false>
tt_status launch_cfg(core3::Params3 &p, hipStream_t s)
{
    auto kern = gemm_bf16_v3_kernel<A_KC, B_KC, OUT_BF16, STAGED, SPREAD, RUNS>;
    constexpr size_t smem = core3::smem_bytes3<64, 2, STAGED>();
    if (ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem) != TT_OK) return TT_EDEVICE;
    hipLaunchKernelGGL(kern, dim3((uint32_t)p.wg_per_xcd * core::kXcds), dim3(core3::kThreads3), smem, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

template <bool A_KC, bool B_KC> tt_status launch_layout(core3::Params3 &p, int out_dtype, bool vec, hipStream_t s)
{
    const bool bf = out_dtype == TT_BF16;
    constexpr bool SPREAD = !A_KC && !B_KC;
    if (vec) return bf ? launch_cfg<A_KC, B_KC, true, true, SPREAD>(p, s) : launch_cfg<A_KC, B_KC, false, true, SPREAD>(p, s);
    return bf ? launch_cfg<A_KC, B_KC, true, false, SPREAD>(p, s) : launch_cfg<A_KC, B_KC, false, false, SPREAD>(p, s);
}

// over runs of K tiles
template <bool A_KC, bool B_KC> tt_status launch_runs(core3::Params3 &p, int out_dtype, hipStream_t s)
{
    constexpr bool SPREAD = !A_KC && !B_KC;
    if (out_dtype == TT_BF16) return launch_cfg<A_KC, B_KC, true, true, SPREAD, true>(p, s);
    return launch_cfg<A_KC, B_KC, false, true, SPREAD, true>(p, s);
}

void set_store(core3::Params3 *p, int out_dtype, int64_t outs)
{
    const int64_t row = (out_dtype == TT_BF16 ? int64_t(2) : int64_t(4)) * p->N;
    p->nts = non_temporal_results(row, row * p->M * outs);
}

} // namespace

// C_s = A_s^T B_s, A_s stored K x M, B_s stored K x N, K up to 512, bf16 result with 16-byte rows.
// TT_EUNSUPPORTED when the engine does not take the product.
tt_status launch_gemm_v5(int count, const void *const *A, const void *const *B, void *const *C, int64_t M, int64_t N,
                         int64_t K, int64_t lda, int64_t ldb, int64_t ldc, int relu, void *stream)
{
    core5::Params5 p;
    const tt_status st = fill_params5(&p, cu_count(), count, A, B, C, M, N, K, lda, ldb, ldc, relu);
    if (st != TT_OK) return st;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (K <= 64) return launch_cfg5<4>(p, s);
    if (K <= 128) return launch_cfg5<8>(p, s);
    return K <= 256 ? launch_cfg5<16>(p, s) : launch_cfg5<32>(p, s);
}

tt_status launch_gemm_v4(int count, const void *const *A, const void *const *B, void *const *C, int64_t M, int64_t N,
                         int64_t K, int64_t lda, int64_t ldb, int64_t ldc, bool a_kc, bool b_kc, int out_dtype, int relu,
                         bool vec, int ksplit, int64_t kchunk, void *stream)
{
    core3::Params3 p;
    const tt_status st = fill_params3(&p, core4::BM4, core4::BN4, 1, 0, count, A, B, C, M, N, K, lda, ldb, ldc, a_kc,
                                      b_kc, relu, ksplit, kchunk);
    if (st != TT_OK) return st;
    set_store(&p, out_dtype, count * ksplit);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (a_kc && b_kc) return launch_layout4<true, true>(p, out_dtype, vec, s);
    if (a_kc && !b_kc) return launch_layout4<true, false>(p, out_dtype, vec, s);
    if (!a_kc && !b_kc) return launch_layout4<false, false>(p, out_dtype, vec, s);
    return launch_layout4<false, true>(p, out_dtype, vec, s);
}

tt_status launch_gemm_v6(int count, const void *const *A, const void *const *B, void *const *C, int64_t M, int64_t N,
                         int64_t K, int64_t lda, int64_t ldb, int64_t ldc, bool a_kc, bool b_kc, int out_dtype, int relu, bool vec,
                         int ksplit, int64_t kchunk, void *stream)
{
    core3::Params3 p;
    const tt_status st = fill_params3(&p, core6::BM6, core6::BN6, 1, 0, count, A, B, C, M, N, K, lda, ldb, ldc, a_kc, b_kc,
                                      relu, ksplit, kchunk);
    if (st != TT_OK) return st;
    set_store(&p, out_dtype, count * ksplit);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (a_kc && b_kc) return launch_layout6<true, true>(p, out_dtype, vec, s);
    if (a_kc && !b_kc) return launch_layout6<true, false>(p, out_dtype, vec, s);
    if (!a_kc && !b_kc) return launch_layout6<false, false>(p, out_dtype, vec, s);
    return launch_layout6<false, true>(p, out_dtype, vec, s);
}

tt_status launch_gemm_v3(int count, const void *const *A, const void *const *B, void *const *C, int64_t M, int64_t N,
                         int64_t K, int64_t lda, int64_t ldb, int64_t ldc, bool a_kc, bool b_kc, int out_dtype, int relu,
                         bool vec, int ksplit, int64_t kchunk, void *stream)
{
    core3::Params3 p;
    const tt_status st = fill_params3(&p, core3::BM3, core3::BN3, 64, cu_count(), count, A, B, C, M, N, K, lda, ldb, ldc, a_kc,
                                      b_kc, relu, ksplit, kchunk);
    if (st != TT_OK) return st;
    set_store(&p, out_dtype, count * ksplit);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (a_kc && b_kc) return launch_layout<true, true>(p, out_dtype, vec, s);
    if (a_kc && !b_kc) return launch_layout<true, false>(p, out_dtype, vec, s);
    if (!a_kc && !b_kc) return launch_layout<false, false>(p, out_dtype, vec, s);
    return launch_layout<false, true>(p, out_dtype, vec, s);
}

// Rows of C of 16-byte vectors; NN, NT and TN (what the layers launch)
tt_status launch_gemm_v3_runs(int nblk, int nred, int parts, const void *const *A, const void *const *B, void *const *C, int64_t M, int64_t N,
                              int64_t K, int64_t lda, int64_t ldb, int64_t ldc, bool a_kc, bool b_kc, int out_dtype, int relu, void *stream)
{
    core3::Params3 p;
    const tt_status st = fill_params3_runs(&p, cu_count(), nblk, nred, parts, A, B, C, M, N, K, lda, ldb, ldc, a_kc, b_kc, relu);
    if (st != TT_OK) return st;
    set_store(&p, out_dtype, nblk * parts);
    if (!a_kc && b_kc) return TT_EUNSUPPORTED;
    // (recorded only once the launch is certain: a refused product is launched, and recorded, shard by shard)
    ProfileScope scope(stream, !a_kc ? TT_K_GEMM_TN : b_kc ? TT_K_GEMM_NT : TT_K_GEMM_NN, nblk * nred, M, N, K,
                       2ull * nblk * nred * ((uint64_t)M * K + (uint64_t)K * N) + (out_dtype == TT_BF16 ? 2ull : 4ull) * nblk * parts * (uint64_t)M * N,
                       2ull * (uint64_t)M * (uint64_t)N * (uint64_t)K * (uint64_t)(nblk * nred));
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (a_kc && b_kc) return launch_runs<true, true>(p, out_dtype, s);
    if (a_kc) return launch_runs<true, false>(p, out_dtype, s);
    return launch_runs<false, false>(p, out_dtype, s);
}

} // namespace tt
