// Launch parameters of the persistent engine (gemm_core3.h), the 256 x 128 engines (gemm_core4.h, gemm_core6.h) and the panel engine (gemm_core5.h): what the
// kernels assume about a product is checked here, on the host, and the grid geometry is derived here.  Shared by the
// launchers and by the host build that checks the kernels' memory accesses, so that both see the same geometry.
#pragma once
#include <cstdint>
#include "gemm_core3.h"
#include "gemm_core4.h"
#include "gemm_core5.h"
#include "tt_internal.h"

namespace tt {

// tile_m x tile_n output tiles, K a multiple of k_tile (1: any); cus: compute units to fill (persistent engine; 0: one workgroup per
// output tile).  Returns TT_EUNSUPPORTED when the engine does not take the product.
inline tt_status fill_params3(core3::Params3 *p, int tile_m, int tile_n, int k_tile, int cus, int count, const void *const *A,
                              const void *const *B, void *const *C, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb,
                              int64_t ldc, bool a_kc, bool b_kc, int relu, int ksplit, int64_t kchunk)
{
    if (K <= 0 || K % k_tile || (ksplit > 1 && kchunk % k_tile) || M < 8 || N < 8) return TT_EUNSUPPORTED;
    if (count * ksplit > 64 || count < 1) return TT_EUNSUPPORTED;
    if ((!a_kc && M % 8) || (!b_kc && N % 8)) return TT_EUNSUPPORTED;
    if (M * K >= (int64_t(1) << 31) || K * N >= (int64_t(1) << 31)) return TT_EUNSUPPORTED; // 32-bit byte offsets
    for (int i = 0; i < 64; ++i) {
        p->A[i] = i < count ? A[i] : nullptr;
        p->B[i] = i < count ? B[i] : nullptr;
        p->C[i] = i < count * ksplit ? C[i] : nullptr;
    }
    p->M = (int32_t)M; p->N = (int32_t)N; p->K = (int32_t)K;
    p->lda = (int32_t)lda; p->ldb = (int32_t)ldb; p->ldc = (int32_t)ldc;
    p->tiles_m = (int32_t)((M + tile_m - 1) / tile_m);
    p->tiles_n = (int32_t)((N + tile_n - 1) / tile_n);
    const int64_t total = (int64_t)p->tiles_m * p->tiles_n * count * ksplit;
    if (total >= (int64_t(1) << 30)) return TT_EUNSUPPORTED;
    p->total = (int32_t)total;
    p->per_xcd = (int32_t)((total + core::kXcds - 1) / core::kXcds);
    p->wg_per_xcd = p->per_xcd;
    if (cus > 0) {
        const int per_xcd_cus = cus / core::kXcds > 0 ? cus / core::kXcds : 1;
        if (per_xcd_cus < p->wg_per_xcd) p->wg_per_xcd = per_xcd_cus;
    }
    p->relu = relu;
    p->nts = 1;
    p->ksplit = ksplit;
    p->kchunk = (int32_t)(ksplit > 1 ? kchunk : K);
    p->nred = p->parts = 1;
    return TT_OK;
}

// Persistent engine over runs of K tiles (RUNS in gemm_core3.h): nblk output blocks of nred shards each (A, B: a block's
// shards one after the other), `parts` runs and results per block.
inline tt_status fill_params3_runs(core3::Params3 *p, int cus, int nblk, int nred, int parts, const void *const *A, const void *const *B,
                                   void *const *C, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, int64_t ldc, bool a_kc,
                                   bool b_kc, int relu)
{
    if (nblk < 1 || nred < 1 || nblk > 64 || nred > 64 || parts < 1 || parts > 64 || nblk * nred > 64 || nblk * parts > 64) return TT_EUNSUPPORTED;
    void *first[64]; // (fill_params3 reads one result per shard)
    for (int i = 0; i < 64; ++i) first[i] = i < nblk * parts ? C[i] : nullptr;
    const tt_status st = fill_params3(p, core3::BM3, core3::BN3, 64, cus, nblk * nred, A, B, first, M, N, K, lda, ldb, ldc, a_kc, b_kc, relu, 1, K);
    if (st != TT_OK) return st;
    const int64_t all = K / 64 * nred; // every run has at least one K tile; products of run and tile numbers fit 32 bits
    if (all < parts || all > (int64_t(1) << 24)) return TT_EUNSUPPORTED;
    for (int i = 0; i < 64; ++i) p->C[i] = first[i];
    const int64_t total = (int64_t)p->tiles_m * p->tiles_n * nblk * parts;
    if (total >= (int64_t(1) << 30)) return TT_EUNSUPPORTED;
    p->total = (int32_t)total;
    p->per_xcd = (int32_t)((total + core::kXcds - 1) / core::kXcds);
    const int per_xcd_cus = cus / core::kXcds > 0 ? cus / core::kXcds : 1;
    p->wg_per_xcd = per_xcd_cus < p->per_xcd ? per_xcd_cus : p->per_xcd;
    p->nred = nred;
    p->parts = parts;
    return TT_OK;
}

// Panel engine: C_s = A_s^T B_s, A_s stored K x M, B_s stored K x N, K up to 512, bf16 results with 16-byte rows
inline tt_status fill_params5(core5::Params5 *p, int cus, int count, const void *const *A, const void *const *B, void *const *C, int64_t M,
                              int64_t N, int64_t K, int64_t lda, int64_t ldb, int64_t ldc, int relu)
{
    if (K < 1 || K > 512 || N < 8 || N % 8 || M < 8 || M % 8 || count < 1 || count > 64) return TT_EUNSUPPORTED;
    if (lda % 8 || ldb % 8 || ldc % 8 || lda < M || ldb < N || ldc < N) return TT_EUNSUPPORTED; // 16-byte chunks and rows
    if (K * lda >= (int64_t(1) << 30) || K * ldb >= (int64_t(1) << 30)) return TT_EUNSUPPORTED; // 32-bit byte offsets
    if (ldc >= (int64_t(1) << 28)) return TT_EUNSUPPORTED; // ... also of the eight rows that a store covers
    for (int i = 0; i < 64; ++i) {
        p->A[i] = i < count ? A[i] : nullptr;
        p->B[i] = i < count ? B[i] : nullptr;
        p->C[i] = i < count ? C[i] : nullptr;
    }
    p->M = (int32_t)M; p->N = (int32_t)N; p->K = (int32_t)K;
    p->lda = (int32_t)lda; p->ldb = (int32_t)ldb; p->ldc = (int32_t)ldc;
    p->panels = (int32_t)((M + core5::PM5 - 1) / core5::PM5);
    p->ntiles = (int32_t)((N + core5::NT5 - 1) / core5::NT5);
    const int64_t total = (int64_t)count * p->panels * p->ntiles;
    if (total >= (int64_t(1) << 30)) return TT_EUNSUPPORTED;
    p->total = (int32_t)total;
    const int64_t resident = (K <= 256 ? 2 : 1) * (int64_t)cus; // two workgroups per CU; one at K = 512
    p->grid = (int32_t)(total < resident ? total : resident);
    p->relu = relu;
    return TT_OK;
}

} // namespace tt
