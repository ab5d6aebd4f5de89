// Shard products that the MFMA tile engines do not take: fp32, or bf16 rows without 16-byte vectors (gemm_small.h).
// One launch covers all shards (Sec. 5.2 step 2 of arXiv 1805.04170).
#include "tt_device.h"
#include <cstdint>
#include "gemm_small.h"
#include "tt_internal.h"

namespace tt {
namespace {

using core::kXcds;

template <bool BF, bool A_KC, bool B_KC, int T, class OFF>
__global__ __launch_bounds__(small::waves_of<T>() * 64, T == 1 ? 2 : 1) void gemm_small_kernel(const small::ParamsS p)
{
    __shared__ __attribute__((aligned(16))) char lds[small::waves_of<T>() * small::lds_per_wave<BF, A_KC, B_KC, T>()];
    small::run_small<BF, A_KC, B_KC, T, OFF>(p, lds);
}

template <bool BF, int T, class OFF> tt_status launch_small_layout(const small::ParamsS &p, bool a_kc, bool b_kc, hipStream_t s)
{
    const dim3 grid(p.per_xcd > 0 ? (uint32_t)p.per_xcd * kXcds : (uint32_t)p.total), block(p.wm * p.wn * p.wk * 64);
    if (a_kc && b_kc) hipLaunchKernelGGL((gemm_small_kernel<BF, true, true, T, OFF>), grid, block, 0, s, p);
    else if (a_kc) hipLaunchKernelGGL((gemm_small_kernel<BF, true, false, T, OFF>), grid, block, 0, s, p);
    else if (b_kc) hipLaunchKernelGGL((gemm_small_kernel<BF, false, true, T, OFF>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((gemm_small_kernel<BF, false, false, T, OFF>), grid, block, 0, s, p);
    return hipGetLastError() == hipSuccess ? TT_OK : TT_EDEVICE;
}

// Block size and the waves' split between K and N (gemm_small.h); count * ksplit outputs of M x N.
template <bool BF> tt_status launch_small(small::ParamsS &p, int count, bool a_kc, bool b_kc, hipStream_t s)
{
    const int64_t outs = (int64_t)count * p.ksplit;
    // 64 x 64 blocks halve what a product reads through L2; they pay once they give every CU a workgroup (bf16, NN: 128 of
    // them, 256 x 2047 x 2047, 26 us against 21.5 with 32 x 32 blocks; 256, 1001 x 1003 x 1007, 18 against 21.6; fp32 32 against 43)
    const bool big_pitch = p.lda >= (1 << 24) || p.ldb >= (1 << 24); // a lane's offset inside a block must fit 32 bits
    const int64_t blocks64 = (int64_t)((p.M + 63) / 64) * ((p.N + 63) / 64) * outs;
    const int T = !big_pitch && p.M > 32 && p.N > 32 && blocks64 >= tuning_int("TT_SMALL_T2", 256) ? 2 : 1;
    // Waves along K: as many as leave each of them two chunks (both on their way at once: a wave alone would not be done
    // sooner with one), while the output blocks alone do not give every CU eight waves.  Four waves at least: what K does
    // not take lies side by side along N, then M.
    const int S = 32 * T, KU = small::chunk_k<BF>(), W = T == 1 ? small::waves_of<1>() : small::waves_of<2>();
    const int64_t chunks = ((int64_t)(p.ksplit > 1 ? p.kchunk : p.K) + KU - 1) / KU;
    p.wk = 1;
    const int64_t blocks = T == 2 ? blocks64 : (int64_t)((p.M + 31) / 32) * ((p.N + 31) / 32) * outs;
    while (p.wk < W && 4 * p.wk <= chunks && blocks * p.wk < 2048) p.wk *= 2;
    p.wn = p.wk <= 2 ? 2 : 1;
    p.wm = p.wk == 1 ? 2 : 1;
    p.tiles_m = (int32_t)(((int64_t)p.M + p.wm * S - 1) / (p.wm * S));
    p.tiles_n = (int32_t)(((int64_t)p.N + p.wn * S - 1) / (p.wn * S));
    const int64_t total = (int64_t)p.tiles_m * p.tiles_n * outs;
    if (total >= (int64_t(1) << 30)) return TT_EUNSUPPORTED;
    p.total = (int32_t)total;
    p.per_xcd = total < 8 * kXcds ? 0 : (int32_t)((total + kXcds - 1) / kXcds); // (a handful of workgroups: any order will do)
    if (big_pitch) return launch_small_layout<BF, 1, uint64_t>(p, a_kc, b_kc, s);
    return T == 2 ? launch_small_layout<BF, 2, uint32_t>(p, a_kc, b_kc, s) : launch_small_layout<BF, 1, uint32_t>(p, a_kc, b_kc, s);
}

} // namespace

// C_s = op(A_s) op(B_s); lda, ldb: elements between rows of the stored matrices; a_kc / b_kc: the operand has K contiguous
tt_status launch_gemm_small(int count, const void *const *A, const void *const *B, void *const *C, int64_t M, int64_t N, int64_t K,
                            int64_t lda, int64_t ldb, bool a_kc, bool b_kc, int in_dtype, int out_dtype, int relu, int ksplit,
                            int64_t kchunk, void *stream)
{
    if (count < 1 || count * ksplit > kMaxShards) return TT_EINVAL;
    small::ParamsS g;
    for (int i = 0; i < kMaxShards; ++i) {
        g.A[i] = i < count ? A[i] : nullptr;
        g.B[i] = i < count ? B[i] : nullptr;
        g.C[i] = i < count * ksplit ? C[i] : nullptr;
    }
    g.M = (int32_t)M; g.N = (int32_t)N; g.K = (int32_t)K;
    g.lda = lda;
    g.ldb = ldb;
    g.ldc = (int32_t)N;
    g.ksplit = ksplit;
    g.kchunk = (int32_t)kchunk;
    g.relu = relu;
    g.out_bf16 = out_dtype == TT_BF16;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    return in_dtype == TT_BF16 ? launch_small<true>(g, count, a_kc, b_kc, s) : launch_small<false>(g, count, a_kc, b_kc, s);
}

} // namespace tt
